"""GPU tests of batches whose members stand at different points of their cycles."""
import numpy as np
import pytest
import torch

import synthetic as sy

pytestmark = pytest.mark.gpu

import gpu_util as gu  # noqa: E402  (an import error fails the run)

# (length, chains, global_every, anchor_every, sweeps before the batch)
MEMBERS = [(20, 3, 0, 1000, 0), (33, 5, 10, 1, 4), (24, 2, 3, 3, 1), (50, 4, 0, 2, 0), (41, 3, 1, 5, 2), (28, 6, 10, 10, 7)]


def _members():
    out = []
    for q, (L, C, every, anchor, _) in enumerate(MEMBERS):
        w = sy.Workload(f"phase{q}", L=L, n_chains=C, total_sweeps=100, window_d=8, global_every=every,
                        anchor_every=anchor, seed=0xfa5e + q, protein_seed=q + 1, noise_seed=q + 2)
        out.append((w, gu.protein(w)[1]))
    return out


def _state(ctx):
    st = ctx.get_state()
    torch.cuda.synchronize()
    return {k: (v.cpu().numpy() if torch.is_tensor(v) else v) for k, v in st.items()}


@pytest.mark.parametrize("plan", [0, 2, 5])
def test_members_out_of_phase_equal_plain_launches(plan):
    """Localized-only, alternating and global-only members with anchors from every sweep to none, each
    at its own sweep: several batch calls one behind the other (whole, uneven, with members that
    stand still), then the members alone again.  The same states as without a batch."""
    from paper_2211_03193_amd import amh
    gu.say("out of phase, plan", plan)
    members = _members()
    calls = [9, [4, 0, 7, 3, 1, 12], 20, [1, 1, 0, 0, 2, 0], 5]
    ctxs = [gu.context(w, y) for w, y in members]
    for ctx, m in zip(ctxs, MEMBERS):
        ctx.sweep(m[4])
    b = amh.Batch(ctxs)
    b.set_plan(plan)
    for n in calls:
        b.sweep(n)
    for ctx in ctxs:   # on the common stream, behind the batch's
        ctx.sweep(2)
    b.sweep(3)
    b.close()
    for q, (ctx, (w, y), m) in enumerate(zip(ctxs, members, MEMBERS)):
        ctx.poll()
        ref = gu.context(w, y)
        ref.sweep(m[4] + sum(n if isinstance(n, int) else n[q] for n in calls) + 5)
        a, z = _state(ctx), _state(ref)
        for k in ("s", "s_best", "v", "counters", "atoms", "t"):
            assert np.array_equal(a[k], z[k]), (q, k)
        ref.close()
        ctx.close()


def test_more_steps_than_the_rings_hold():
    """Anchors after every sweep beside long runs, 150 steps of one member in one call: more than
    the staging buffers of a stream hold at once."""
    from paper_2211_03193_amd import amh
    gu.say("out of phase, many steps")
    ws = [sy.Workload(f"long{q}", L=12 + q, n_chains=2, total_sweeps=150, window_d=4, global_every=0,
                      anchor_every=a, seed=0x10e + q, protein_seed=q + 1, noise_seed=q + 2)
          for q, a in enumerate((1, 1000, 2))]
    ys = [gu.protein(w)[1] for w in ws]
    ctxs = [gu.context(w, y) for w, y in zip(ws, ys)]
    b = amh.Batch(ctxs)
    b.sweep(150)
    for ctx, w, y in zip(ctxs, ws, ys):
        ref = gu.context(w, y)
        ref.sweep(150)
        a, z = _state(ctx), _state(ref)
        assert all(np.array_equal(a[k], z[k]) for k in ("s", "s_best", "v", "counters", "atoms"))
        ref.close()
    b.close()
    for ctx in ctxs:
        ctx.close()
