"""The launch rules that the host applies to a configuration, without a GPU."""
import os
import shutil
import subprocess

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
