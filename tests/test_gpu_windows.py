"""GPU tests of localized sweeps whose window is wider than the chain."""
import numpy as np
import pytest

import synthetic as sy

pytestmark = pytest.mark.gpu

import gpu_util as gu  # noqa: E402  (an import error fails the run)


@pytest.mark.parametrize("G", [1, 2, 4])
def test_windows_wider_than_the_chain(G):
    """Radii up to the largest 32-bit number, one after the other in a cascade: every proposal
    as with radii of twice the chain, and as the oracle's."""
    L, C, n = 21, 5, 15
    w = sy.Workload(f"wide-{G}", L=L, n_chains=C, total_sweeps=n, window_d=2 * L, cascade=(2 * L, 6, 2 * L),
                    global_every=0, anchor_every=15, seed=0x31d, protein_seed=8, noise_seed=9)
    s_ref, y = gu.protein(w)
    rng = np.random.Generator(np.random.PCG64(3))
    s0 = sy._wrap(s_ref[None] + 0.2 * rng.standard_normal((C, 2 * L)))
    out = []
    for radii in ((2 * L, 2 * L, 6, 2 * L), (2**31 - 1, 10**6, 6, 2**30)):
        gu.say("windows wider than the chain", G, radii)
        wide = w.replace(window_d=radii[0], cascade=radii[1:])
        ctx = gu.context(wide, y, s0=s0, chains_per_group=G, waves_per_group=4)
        tr = gu.traced_run(ctx, [0, 4], n)
        st = ctx.get_state()
        ctx.close()
        for slot, chain in enumerate((0, 4)):
            rc, rep, _ = gu.replay_chain(w, y, tr, slot, chain, s0[chain])
            assert rc == 0 and rep["n_de_fail"] == 0 and rep["n_logic_fail"] == 0, (radii, rep)
        out.append([st[k].cpu().numpy() for k in ("s", "v", "counters")] + [tr["dE"]])
    assert all(np.array_equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("bin_w", [1e19, 1e30])
def test_bins_wider_than_any_chain(bin_w):
    """Every pair below the first knot, where the energy is flat: nothing a proposal does changes
    it, localized or global, and absent residues of the last tiles are no pairs."""
    w = sy.Workload("bins", L=13, n_chains=3, total_sweeps=4, window_d=6, global_every=2, anchor_every=2, seed=0xb1,
                    protein_seed=5, noise_seed=6)
    _, y = gu.protein(w)
    gu.say("bins of", bin_w)
    ctx = gu.context(w, y, bin_w=bin_w, d_min=0.0)
    tr = gu.traced_run(ctx, [0, 2], 4)
    V, _, _ = ctx.energy()
    V = V.cpu().numpy()
    ctx.close()
    assert np.all(tr["dE"] == 0.0) and np.all(tr["acc"] == 1)
    first = np.asarray(y, dtype=np.float32)[:, 0].astype(np.float64).sum()
    assert V == pytest.approx(np.full(3, first), rel=1e-12)
    assert tr["anchor"][:2, :2] == pytest.approx(np.full((2, 2), first), rel=1e-12)


@pytest.mark.parametrize("G", [1, 2, 4])
@pytest.mark.parametrize("d, cascade", [(8, ()), (12, (4, 30)), (14, ()), (36, (2,))])
def test_walls_cost_no_digits_of_an_energy_change(G, d, cascade):
    """Neighbours in the chain held below the first knot, where their energy is flat: with 1e15
    there instead of 2, every localized proposal has the same energy change, bit for bit, and
    without the wall it is the oracle's."""
    L, C, n = 40, 5, 14
    w = sy.Workload("walls", L=L, n_chains=C, total_sweeps=n, window_d=d, cascade=cascade, global_every=0,
                    anchor_every=100, seed=0x3a11, protein_seed=8, noise_seed=9, d_min=6.5)
    _, y = gu.protein(w)
    s_ref = sy.reference_torsions(L, 8)
    rng = np.random.Generator(np.random.PCG64(4))
    s0 = sy._wrap(s_ref[None] + 0.2 * rng.standard_normal((C, 2 * L)))
    i = np.arange(L - 1)
    rows = i * L - i * (i + 1) // 2   # of the pairs (i, i + 1)
    out = []
    for wall in (2.0, 1e15):
        gu.say("walls of", wall, "in windows of", d, cascade, "G", G)
        table = np.array(y)
        table[rows, :-1] = wall
        table[rows, -1] = 3.0
        ctx = gu.context(w, table, s0=s0, chains_per_group=G, waves_per_group=4)
        tr = gu.traced_run(ctx, [0, 4], n)
        st = ctx.get_state()
        ctx.close()
        if wall == 2.0:
            for slot, chain in enumerate((0, 4)):
                rc, rep, _ = gu.replay_chain(w, table, tr, slot, chain, s0[chain])
                assert rc == 0 and rep["n_de_fail"] == 0 and rep["n_logic_fail"] == 0, rep
        out.append([tr["dE"], tr["acc"], st["s"].cpu().numpy(), st["counters"].cpu().numpy()])
    assert all(np.array_equal(a, b) for a, b in zip(*out))
