"""GPU tests of the gradient's workgroup shapes: long chains, one workgroup a compute unit."""
import numpy as np
import pytest
import torch

import oracle
import synthetic as sy

pytestmark = pytest.mark.gpu

import gpu_util as gu  # noqa: E402  (an import error fails the run)


@pytest.mark.parametrize("L", [470, 471, 540, 830, 970])
def test_grad_of_long_chains_at_every_workgroup_size(L):
    """Two workgroups of 4 wavefronts a compute unit, one of 8 with long and with short lists,
    one of 4.  The same bits for few and for many conformations, energies as the oracle's."""
    gu.say("gradients of long chains, L", L)
    w = sy.CFG1.replace(L=L, n_chains=1, protein_seed=L, noise_seed=L + 1)
    s_ref, y = gu.protein(w)
    ctx = gu.context(w, y)
    s = np.stack([s_ref, np.tile([-1.05, -0.79], L)])
    cfg = oracle.make_cfg(w)
    y32 = y.astype(np.float32).astype(np.float64)
    ref = np.array([oracle.energy(cfg, y32, x) for x in s])
    first = None
    for B in (2, 260, 520):
        V, g = ctx.grad(torch.from_numpy(np.tile(s, (B // 2, 1))).to(gu.DEV))
        V, g = V.cpu().numpy().reshape(-1, 2), g.cpu().numpy().reshape(-1, 2, 2 * L)
        if first is None:
            first = V[0], g[0]
            assert V[0] == pytest.approx(ref, rel=1e-12)
        assert np.array_equal(V, np.broadcast_to(first[0], V.shape)), B
        assert np.array_equal(g, np.broadcast_to(first[1], g.shape)), B
    ctx.close()


@pytest.mark.parametrize("L", [8, 9, 64, 90, 128])
def test_grad_of_coils(L):
    """Coils with every pair inside the last knot: a tile to a wavefront and tiles shared by 8, 4
    and 2 wavefronts; with 128 residues and four wavefronts the list holds two of the three tiles at a
    time.  The same bits at every size, energies as the oracle's."""
    gu.say("gradients of coils, L", L)
    w = sy.CFG1.replace(L=L, n_chains=1, protein_seed=L, noise_seed=L + 1)
    s_ref, y = gu.protein(w)
    ctx = gu.context(w, y)
    s = np.stack([np.tile(np.deg2rad([-120.0, -40.0]), L), s_ref])
    cb = oracle.cb(s[0]).reshape(L, 3)
    assert np.linalg.norm(cb[:, None] - cb[None], axis=-1).max() < 20.25
    cfg = oracle.make_cfg(w)
    y32 = y.astype(np.float32).astype(np.float64)
    ref = np.array([oracle.energy(cfg, y32, x) for x in s])
    first = None
    for B in (1026, 2, 260, 514):
        V, g = ctx.grad(torch.from_numpy(np.tile(s, (B // 2, 1))).to(gu.DEV))
        V, g = V.cpu().numpy().reshape(-1, 2), g.cpu().numpy().reshape(-1, 2, 2 * L)
        if first is None:
            first = V[0], g[0]
            assert V[0] == pytest.approx(ref, rel=1e-12)
        assert np.array_equal(V, np.broadcast_to(first[0], V.shape)), B
        assert np.array_equal(g, np.broadcast_to(first[1], g.shape)), B
    ctx.close()
