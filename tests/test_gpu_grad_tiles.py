"""GPU tests of the gradient's pair tiles, lists and workgroup sizes."""
import numpy as np
import pytest
import torch

import oracle
import synthetic as sy

pytestmark = pytest.mark.gpu

import gpu_util as gu  # noqa: E402  (an import error fails the run)


@pytest.mark.parametrize("L", [2, 63, 64, 65, 128, 129, 200])
def test_grad_at_every_workgroup_size(L):
    """One tile, whole and ragged last tiles; one, two and more conformations a compute unit
    (workgroups of 8, 4 and, up to 128 residues, 2 wavefronts, with lists of different
    lengths).  Compact, extended and helical conformations: the same bits at every size
    (the gradients of few conformations are held against the oracle's in test_gpu_grad.py),
    energies as the oracle's."""
    gu.say("gradients by workgroup size, L", L)
    w = sy.CFG1.replace(L=L, n_chains=1, protein_seed=L, noise_seed=L + 1)
    s_ref, y = gu.protein(w)
    ctx = gu.context(w, y)
    helix = np.tile([-1.05, -0.79], L)
    s = np.stack([s_ref, np.full(2 * L, np.pi), helix])
    cfg = oracle.make_cfg(w)
    y32 = y.astype(np.float32).astype(np.float64)
    ref = np.array([oracle.energy(cfg, y32, x) for x in s])
    first = None
    for B in (3, 258, 513, 1026):
        V, g = ctx.grad(torch.from_numpy(np.tile(s, (B // 3, 1))).to(gu.DEV))
        V, g = V.cpu().numpy().reshape(-1, 3), g.cpu().numpy().reshape(-1, 3, 2 * L)
        if first is None:
            first = V[0], g[0]
            assert V[0] == pytest.approx(ref, rel=1e-12)
        assert np.array_equal(V, np.broadcast_to(first[0], V.shape)), B
        assert np.array_equal(g, np.broadcast_to(first[1], g.shape)), B
    ctx.close()


def test_grad_of_the_longest_helix():
    """1024 residues: coordinates that leave room for short lists only, which the tiles on a
    helix's diagonal (over 800 pairs inside the last knot) overflow.  Tolerance: coordinates of
    two NeRFs differ by 3 L eps R = 1e-9 A (R = 1540 A), a force by that over the bin width,
    2e-9 of it, and the forces of some 30 pairs cancel in a residue's: 1e-7 of the largest."""
    L = 1024
    gu.say("gradient of a helix of", L)
    w = sy.CFG1.replace(L=L, n_chains=1, protein_seed=3, noise_seed=4)
    _, y = gu.protein(w)
    ctx = gu.context(w, y)
    s = np.tile([-1.05, -0.79], L)
    V, g = ctx.grad(torch.from_numpy(s[None]).to(gu.DEV))
    ctx.close()
    Vo, go = oracle.grad(oracle.make_cfg(w), y.astype(np.float32).astype(np.float64), s)
    assert V.item() == pytest.approx(Vo, rel=1e-12)
    assert np.abs(g[0].cpu().numpy() - go).max() <= 1e-7 * np.abs(go).max()
