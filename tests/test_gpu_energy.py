"""GPU tests of the energy kernel's workgroup sizes, tile fold and pair queues."""
import numpy as np
import pytest
import torch

import oracle
import synthetic as sy

pytestmark = pytest.mark.gpu

import gpu_util as gu  # noqa: E402  (an import error fails the run)


@pytest.mark.parametrize("L", [2, 8, 9, 17, 24, 65, 130])
def test_energy_at_every_workgroup_size(L):
    """One, two and more conformations a compute unit (workgroups of 16, 8 and 4 wavefronts),
    odd and even numbers of 8-residue blocks, compact and extended conformations (full and
    empty pair queues): against the oracle, and the same bits at every size."""
    gu.say("energies by workgroup size, L", L)
    w = sy.CFG1.replace(L=L, n_chains=1, protein_seed=L, noise_seed=L + 1)
    s_ref, y = gu.protein(w)
    ctx = gu.context(w, y)
    s = np.stack([s_ref, sy.random_torsions(2 * L, 7), np.full(2 * L, np.pi)])
    cfg = oracle.make_cfg(w)
    y32 = y.astype(np.float32).astype(np.float64)
    ref = np.array([oracle.energy(cfg, y32, x) for x in s])
    first = None
    for B in (3, 258, 513, 1026):
        V, _, _ = ctx.energy(torch.from_numpy(np.tile(s, (B // 3, 1))).to(gu.DEV))
        V = V.cpu().numpy().reshape(-1, 3)
        assert np.array_equal(V, np.broadcast_to(V[0], V.shape)), B
        if first is None:
            first = V[0]
            assert V[0] == pytest.approx(ref, rel=1e-9)
        assert np.array_equal(V[0], first), B
    ctx.close()
