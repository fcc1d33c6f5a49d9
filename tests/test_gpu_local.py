"""GPU tests of the localized-sweep kernel at the edges of its pair deals and launch shapes."""
import numpy as np
import pytest

import synthetic as sy

pytestmark = pytest.mark.gpu

import gpu_util as gu  # noqa: E402  (an import error fails the run)


@pytest.mark.parametrize("L, d, cascade", [
    (2, 4, ()), (3, 12, ()), (5, 0, ()), (9, 2, ()), (24, 12, ()), (25, 12, ()), (40, 14, ()),
    (40, 30, ()), (41, 32, ()), (70, 62, ()), (66, 64, ()), (140, 128, ()), (140, 132, ()), (30, 200, ()),
    (60, 12, (4, 34, 14)),
])
def test_localized_sweeps_at_deal_edges(L, d, cascade):
    """Windows of d residues around the deals of a chain's pairs to its 16, 32 or 64 lanes: a
    lane a pair and no longer (d = 12, 14), a lane a column and no longer (d = 30 to 132), a
    window as long as the chain, a quarter of it (24 and 25 residues) and wider, and several
    widths in turn; one and several wavefronts, ragged last workgroups.  Every proposal of two
    chains against the oracle, and the same final state in every launch shape."""
    w = sy.Workload(f"deal-L{L}-d{d}", L=L, n_chains=5, total_sweeps=5, window_d=d, cascade=cascade, global_every=0,
                    anchor_every=3, seed=0x10c + L + d, protein_seed=L, noise_seed=L + 1)
    s_ref, y = gu.protein(w)
    rng = np.random.Generator(np.random.PCG64(L))
    s0 = sy._wrap(s_ref[None] + 0.2 * rng.standard_normal((5, 2 * L)))
    first = None
    for G, W in ((0, 0), (1, 1), (1, 3), (2, 4), (4, 4), (4, 8)):
        gu.say("localized sweeps", L, d, (G, W))
        ctx = gu.context(w, y, s0=s0, chains_per_group=G, waves_per_group=W)
        tr = gu.traced_run(ctx, [0, 4], 5, chunk=5)
        st = ctx.get_state()
        ctx.close()
        for slot, chain in enumerate((0, 4)):
            rc, rep, s_end = gu.replay_chain(w, y, tr, slot, chain, s0[chain])
            assert rc == 0 and rep["n_de_fail"] == 0 and rep["n_logic_fail"] == 0, ((G, W), rep)
            assert np.abs(s_end - st["s"][chain].cpu().numpy()).max() <= 1e-12
        out = [st[k].cpu().numpy() for k in ("s", "v", "counters")]
        if first is None:
            first = out
        assert all(np.array_equal(a, b) for a, b in zip(first, out)), (G, W)


@pytest.mark.parametrize("C", [256, 257, 512, 513, 1025, 1281, 1540])
def test_localized_launches_by_chain_count(C):
    """Chain counts around the sizes where a context's localized launches change (1, 2 or 4
    chains a workgroup, a second launch for the chains beyond whole rounds): the last chains
    against the oracle, and every chain as in single-chain workgroups."""
    w = sy.Workload(f"launches-C{C}", L=12, n_chains=C, total_sweeps=6, window_d=4, global_every=3, anchor_every=3,
                    seed=0x3a0 + C, protein_seed=5, noise_seed=6)
    s_ref, y = gu.protein(w)
    rng = np.random.Generator(np.random.PCG64(C))
    s0 = sy._wrap(s_ref[None] + 0.3 * rng.standard_normal((C, 2 * w.L)))
    out = []
    for G, W in ((0, 0), (1, 4)):
        gu.say("localized launches", C, (G, W))
        ctx = gu.context(w, y, s0=s0, chains_per_group=G, waves_per_group=W)
        chains = [0, C - 2, C - 1]
        tr = gu.traced_run(ctx, chains, 6)
        st = ctx.get_state()
        ctx.close()
        for slot, chain in enumerate(chains):
            rc, rep, s_end = gu.replay_chain(w, y, tr, slot, chain, s0[chain])
            assert rc == 0 and rep["n_de_fail"] == 0 and rep["n_logic_fail"] == 0, ((G, W), rep)
            assert np.abs(s_end - st["s"][chain].cpu().numpy()).max() <= 1e-12
        out.append([st[k].cpu().numpy() for k in ("s", "v", "counters")])
    assert all(np.array_equal(a, b) for a, b in zip(*out))
