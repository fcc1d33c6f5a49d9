"""GPU test of energies and anchors at the lengths where their workgroups' sizes change."""
import numpy as np
import pytest
import torch

import oracle
import synthetic as sy

pytestmark = pytest.mark.gpu

import gpu_util as gu  # noqa: E402  (an import error fails the run)


@pytest.mark.parametrize("L", [2, 15, 16, 17, 40, 41])
def test_short_chains_by_workgroup_size(L):
    """2, 4 and up to 16 wavefronts a conformation (up to 16, 40 and beyond): energies as the
    oracle's and the same bits for any number of conformations, and an anchor's energy after
    a sweep that accepts nothing the start's."""
    gu.say("short chains, L", L)
    w = sy.CFG1.replace(L=L, n_chains=2, total_sweeps=1, global_every=0, anchor_every=1, sigma_deg=0.0, protein_seed=L,
                        noise_seed=L + 1)
    s_ref, y = gu.protein(w)
    s = np.stack([s_ref, sy.random_torsions(2 * L, 7)])
    cfg = oracle.make_cfg(w)
    ref = np.array([oracle.energy(cfg, y.astype(np.float32).astype(np.float64), x) for x in s])
    ctx = gu.context(w, y, s0=s)
    ctx.sweep(1)
    ctx.poll()
    st = ctx.get_state()
    first = st["v"][:, 0].cpu().numpy()
    assert first == pytest.approx(ref, rel=1e-9)
    for B in (2, 300, 600, 1100):
        V, _, cb = ctx.energy(torch.from_numpy(np.tile(s, (B // 2, 1))).to(gu.DEV), want_cb=True)
        assert np.array_equal(V.cpu().numpy(), np.tile(first, B // 2)), B
        cb = cb.cpu().numpy().reshape(-1, 2, L, 3)
        assert np.array_equal(cb, np.broadcast_to(st["atoms"][:, :, 3].cpu().numpy().astype(np.float32), cb.shape)), B
    ctx.close()
