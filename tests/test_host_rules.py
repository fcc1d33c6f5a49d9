"""The launch rules that the host applies to a configuration, without a GPU."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    exe = str(tmp_path_factory.mktemp("rules") / "probe")
    subprocess.run([hipcc, "-std=c++17", "--offload-arch=gfx950", "--offload-host-only",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2211_03193_amd", "csrc"),
                    os.path.join(HERE, "host_rules_probe.cpp"), "-o", exe], check=True)
    return lambda *a: subprocess.run([exe, *map(str, a)], check=True, capture_output=True, text=True).stdout.split()


@pytest.mark.parametrize("L", [2, 3, 64, 1024])
def test_half_window_is_at_most_the_chain(rule, L):
    """A localized kernel's loops run over the half-width and its wait target adds two of them
    to a residue: a radius of any size gives the window of one as wide as the chain, and no
    narrower one changes."""
    for d in (0, 1, 2, 7, 2 * L - 3, 2 * L - 2, 2 * L - 1, 2 * L, 10**6, 2**30, 2**31 - 1):
        h = int(rule("half_window", d, L)[0])
        assert h <= L - 1
        for c in range(L):   # the same window as the radius asks for
            assert max(0, c - h) == max(0, c - d // 2) and min(L - 1, c + h) == min(L - 1, c + d // 2)


@pytest.mark.parametrize("d_min, bin_w, n_bins", [(2.0, 0.5, 37), (0.0, 1e3, 64), (-40.0, 1.0, 37), (0.0, 1e18, 4),
                                                  (1e19, 1.0, 37), (-1e300, 1e30, 37), (0.0, 1e300, 64)])
def test_absent_residues_lie_beyond_the_last_knot(rule, d_min, bin_w, n_bins):
    """The squared distances at which the global kernel places absent rows (-1e18 A on every
    axis) and columns (+1e18 A): from each other and from residues of a chain, whatever the
    configured bins, and no pair of a chain of 1024 residues is taken out by the bound."""
    d2 = np.float32(rule("last_knot2", d_min, bin_w, n_bins)[0])
    far = np.float32(1e18)
    for x in (0.0, 5e3, -5e3):
        a = np.float32(x) - far
        assert not a * a + a * a + a * a < d2
    assert not np.float32(np.inf) < d2
    knot = d_min + bin_w * (n_bins - 0.5)
    assert d2 == np.float32(knot * knot) if abs(knot) < 1e15 else d2 > 1e8


@pytest.mark.parametrize("L", [2, 3, 300, 1024])
@pytest.mark.parametrize("every", [0, 1])
def test_a_launch_counts_its_accepted_proposals_in_32_bits(rule, L, every):
    """The longest run of sweeps of one kind without an anchor that a configuration allows: a
    launch has fewer proposals a chain than a 32-bit counter holds, and the runs follow on."""
    end = 2**32 - 1
    t = 0
    for _ in range(3):
        e = int(rule("run_end", L, every, every, 2**31 - 1, t, end)[0])
        assert t < e and (e - t) * 2 * L < 2**31
        t = e


def test_runs_end_at_anchors_and_kinds(rule):
    """Cycles of ten with two global sweeps, anchors every three sweeps."""
    ends, t = [], 0
    while t < 20:
        t = int(rule("run_end", 50, 10, 2, 3, t, 20)[0])
        ends.append(t)
    assert ends == [3, 6, 8, 9, 10, 12, 15, 18, 20]


@pytest.mark.parametrize("L", [2, 40, 300, 1024])
@pytest.mark.parametrize("h", [0, 1, 6, 7, 100, 1023])
def test_carried_energies_are_exact_counts(rule, L, h):
    """The largest table deviation at which localized sweeps may carry their energy along: the
    changed pairs of any proposal (rows and columns that part the window) and the carries (2h + 1),
    each 1.25 times that, stay below 2^53 multiples of 2^-30; a wall does not."""
    h = min(h, L - 1)
    most = max(((p - max(0, c - h)) * (min(L - 1, c + h) - p + 1) for c in range(L) for p in (c, c + 1)), default=0)
    pairs = most + 2 * h + 1
    for dev in (0.0, 20.0, 2.0**23 / pairs / 1.31, 2.0**23 / pairs / 1.25, 1e15, 3e38):
        exact = rule("carry", 4, h, L, repr(float(np.float32(dev))))[1] == "1"
        assert not exact or pairs * 1.25 * dev * 2.0**30 < 2.0**53
        assert exact or dev >= 2.0**23 / pairs / 3.0   # (no more than the window's corners given away)


@pytest.mark.parametrize("G", [1, 2, 4])
def test_every_half_width_has_a_way(rule, G):
    """The rule's quotients over all half-widths up to the chain's length, the shortest and the
    longest chains: an answer, and the narrow windows of short chains summed afresh."""
    for L in (2, 3, 32, 99, 100, 1024):
        for h in {0, 1, 2, 6, 7, 8, 15, 16, 31, 32, 33, 63, 64, 65, 200, 1023}:
            if h <= L - 1:
                pays = rule("carry", G, h, L, 20.0)[0] == "1"
                assert not pays or L >= 24


def test_accepted_shapes_fit_the_launches(rule):
    """Every length and shape (chains, wavefronts) that the admission rule accepts, and the automatic
    shapes: what the localized and the global launches take fits a workgroup's 160 KiB."""
    import ctypes

    from paper_2211_03193_amd import amh
    lib = ctypes.CDLL(amh.LIB_PATH)
    names = {k: f"_ZN3amh{len(k)}{k}Eiii" for k in ("sweep_lds_bytes", "local_lds_bytes", "global_lds_bytes")}
    f = {}
    for k, n in names.items():
        f[k] = getattr(lib, n)
        f[k].argtypes, f[k].restype = [ctypes.c_int] * 3, ctypes.c_size_t
    limit = 160 * 1024
    for L in range(2, 1025):
        for G in (1, 2, 4):
            for W in range(G, 9):
                if f["sweep_lds_bytes"](G, L, W) > limit:
                    continue
                nw = 1
                while 2 * nw * G <= W and nw < 16:
                    nw *= 2
                assert f["local_lds_bytes"](G, L, 12) <= limit, (G, L, W)
                assert f["global_lds_bytes"](G, L, nw) <= limit, (G, L, W)
        # automatic: one chain with up to 16 wavefronts, two with two each
        assert f["sweep_lds_bytes"](1, L, 4) <= limit and f["global_lds_bytes"](1, L, 16) <= limit, L
        if f["sweep_lds_bytes"](4, L, 8) <= limit:
            assert f["global_lds_bytes"](2, L, 2) <= limit, L


def test_benchmark_counts_by_the_same_rule(rule):
    """The benchmark's copy of the rule, which its work counts use."""
    import bench
    for G in (1, 2, 4):
        for h in (1, 2, 4, 6, 7, 8, 9, 10, 15, 18, 30):
            for L in (20, 40, 64, 100, 300, 400):
                if h < L:
                    assert bench.carry_pays(G, h, L) == (rule("carry", G, h, L, 20.0)[0] == "1"), (G, h, L)
