"""GPU tests of the pipelined localized sweeps and of the global kernel's widest workgroups."""
import numpy as np
import pytest
import torch

import synthetic as sy

pytestmark = pytest.mark.gpu

import gpu_util as gu  # noqa: E402  (an import error fails the run)


def _around(s_ref, C, noise, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    return sy._wrap(s_ref[None] + noise * rng.standard_normal((C, len(s_ref))))


def _replayed(w, y, s0, sweeps, chains, **shape):
    """The state and trace of one call of `sweeps` sweeps, every proposal of two chains replayed."""
    ctx = gu.context(w, y, s0=s0, **shape)
    tr = gu.traced_run(ctx, chains, sweeps)
    st = ctx.get_state()
    ctx.close()
    for slot, chain in enumerate(chains):
        rc, rep, s_end = gu.replay_chain(w, y, tr, slot, chain, s0[chain])
        assert rc == 0 and rep["n_de_fail"] == 0 and rep["n_logic_fail"] == 0, (shape, rep)
        assert np.abs(s_end - st["s"][chain].cpu().numpy()).max() <= 1e-12
    return [st[k].cpu().numpy() for k in ("s", "v", "counters", "atoms")]


@pytest.mark.parametrize("L, d, cascade", [(18, 6, ()), (26, 12, (2, 20)), (64, 30, ()), (70, 8, (36, 14))])
def test_more_sweeps_in_a_run_than_wavefronts(L, d, cascade):
    """A run of 40 localized sweeps in one launch, so that each of its 12 wavefronts takes a second,
    a third and some a fourth, on progress counters that are counted on; one radius and several
    in turn, energy changes summed afresh and carried (d = 30, 36).  Every proposal of two of 5
    chains against the oracle, the same state for 1, 2 and 4 chains a workgroup."""
    w = sy.Workload(f"pipeline-{L}-{d}", L=L, n_chains=5, total_sweeps=40, window_d=d, cascade=cascade, global_every=0,
                    anchor_every=40, seed=0x9e1 + L, protein_seed=L, noise_seed=L + 1)
    s_ref, y = gu.protein(w)
    s0 = _around(s_ref, 5, 0.2, L)
    out = []
    for G in (1, 2, 4):
        gu.say("40 localized sweeps in a run", L, d, cascade, "G", G)
        out.append(_replayed(w, y, s0, 40, (0, 4), chains_per_group=G, waves_per_group=4))
    for other in out[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(out[0], other))


@pytest.mark.parametrize("L", [257, 263, 321])
def test_sixteen_wavefronts_a_chain(L):
    """Chains just past 256 residues, few enough for a unit each: workgroups of 16 wavefronts, of which
    most own no chunk of 64 residues, last tiles of 1, 7 and 1 residues.  Every proposal of two
    chains against the oracle, and the same state as with 8 and 4 wavefronts."""
    w = sy.Workload(f"wide-{L}", L=L, n_chains=3, total_sweeps=2, window_d=4, global_every=1, anchor_every=2,
                    seed=0x16 + L, protein_seed=L, noise_seed=L + 1)
    s_ref, y = gu.protein(w)
    s0 = _around(s_ref, 3, 0.1, L)
    out = []
    for W in (0, 8, 4):
        gu.say("global sweeps", L, "W", W)
        ctx = gu.context(w, y, s0=s0, chains_per_group=0 if W == 0 else 1, waves_per_group=W)
        if W == 0:
            assert ctx.info()["global_waves_per_group"] == 16
        ctx.close()
        shape = {} if W == 0 else {"chains_per_group": 1, "waves_per_group": W}
        out.append(_replayed(w, y, s0, 2, (0, 2), **shape))
    for other in out[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(out[0], other))


def test_short_members_in_workgroups_of_sixteen_wavefronts():
    """A batch of two short proteins and a long one, which sets 16 wavefronts a chain for all: the
    same states as in launches of their own."""
    from paper_2211_03193_amd import amh
    gu.say("batch of lengths 270, 20 and 9")
    ws = [sy.Workload(f"mix{L}", L=L, n_chains=3, total_sweeps=8, window_d=6, global_every=2, anchor_every=2,
                      seed=0x3c + L, protein_seed=L, noise_seed=L + 1) for L in (270, 20, 9)]
    ys = [gu.protein(w)[1] for w in ws]
    ctxs = [gu.context(w, y) for w, y in zip(ws, ys)]
    b = amh.Batch(ctxs)
    b.sweep(4)
    for ctx, w, y in zip(ctxs, ws, ys):
        ref = gu.context(w, y)
        ref.sweep(4)
        a, z = ctx.get_state(), ref.get_state()
        for k in ("s", "s_best", "v", "counters", "atoms"):
            assert torch.equal(a[k], z[k]), (w.L, k)
        ref.close()
    b.close()
    for ctx in ctxs:
        ctx.close()
