"""GPU tests of the global-sweep kernel at the edges of its tiles and launch shapes."""
import numpy as np
import pytest

import synthetic as sy

pytestmark = pytest.mark.gpu

import gpu_util as gu  # noqa: E402  (an import error fails the run)


@pytest.mark.parametrize("L", [2, 3, 7, 8, 9, 10, 15, 17, 23, 63, 64, 66, 130])
def test_global_sweeps_at_tile_edges(L):
    """Lengths around the 8-residue tiles, the 64-residue chunks and the 21-residue
    backbone window (last tiles of 1 to 8 residues, more and fewer chunks than
    wavefronts): every proposal of two chains of a ragged last workgroup against the
    oracle, and the same final torsions and counters in every launch shape."""
    w = sy.Workload(f"tiles-L{L}", L=L, n_chains=5, total_sweeps=4, window_d=4, global_every=1, anchor_every=2,
                    seed=0x910 + L, protein_seed=L, noise_seed=L + 1)
    s_ref, y = gu.protein(w)
    rng = np.random.Generator(np.random.PCG64(L))
    s0 = sy._wrap(s_ref[None] + 0.2 * rng.standard_normal((5, 2 * L)))
    first = None
    for G, W in ((0, 0), (1, 1), (1, 3), (1, 4), (2, 4), (2, 7), (4, 8)):
        gu.say("global sweeps", L, (G, W))
        ctx = gu.context(w, y, s0=s0, chains_per_group=G, waves_per_group=W)
        tr = gu.traced_run(ctx, [0, 4], 4, chunk=3)
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
