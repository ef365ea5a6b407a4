"""The reduce's slice table where its two searches can go wrong: a thread per boundary and
teams of lanes that find one or several in turn, told apart by the number of tiles and the
planned length of a slice; lists shorter than a line, empty ones, ones that begin anywhere in a line, clustered
ones whose guesses miss, ones that reach out of their region, regions narrower than the
widest.  The line arithmetic itself is checked on the CPU."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_line_search_matches_std_lower_bound(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = tmp_path / "line_search_check"
    subprocess.run([gxx, "-O2", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2201_07598_amd", "csrc"),
                    os.path.join(ROOT, "tests", "cabi", "line_search_check.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert " 0 disagreements" in out.stdout


def contribution(rng, lo, hi, kind):
    width = hi - lo
    if width == 0 or kind == 0:
        return np.zeros(0, np.uint32)
    if kind == 1:                                        # shorter than a line
        at = rng.integers(0, width, int(rng.integers(1, 40)))
    elif kind == 2:                                      # clustered: guesses miss
        at = int(rng.integers(0, width)) + rng.integers(0, max(2, width // 50), 500)
    elif kind == 3:                                      # both ends of the region
        at = np.concatenate([[0, width - 1], rng.integers(0, width, 30)])
    else:
        at = rng.integers(0, width, int(rng.integers(30, 900)))
    out = np.unique(at[at < width]).astype(np.int64) + lo
    if kind == 5:                                        # beyond the region on both sides
        out = np.concatenate([np.arange(max(lo - 40, 0), lo), out, np.arange(hi, hi + 40)])
    return out.astype(np.uint32)


def picks(rng, lo, hi, m):
    return (np.unique(rng.integers(0, max(hi - lo, 1), min(m, hi - lo))) + lo).astype(np.uint32)


# Planned slices of 99 entries in 218 tiles (teams, with two boundaries in turn and one), of
# 295 in 28 (teams), of 55 in 32, 6 in 34 and in 3 tiles (threads).
@pytest.mark.gpu
@pytest.mark.parametrize("B,P,width,share", [(44, 64, 2_000_000, 0.5), (4, 64, 2_000_000, 0.5), (30, 33, 300_000, 0.6),
                                             (30, 64, 500_000, 0.2), (3, 700, 400_000, 0.3), (600, 9, 9_000, 0.9)])
@pytest.mark.parametrize("lead", [0, 3])
def test_slice_tables(B, P, width, share, lead):
    from tests.test_gpu_reduce_tiles import run_batch
    rng = np.random.default_rng(B + P + lead)
    regions = []
    for b in range(B):
        lo = int(rng.integers(100, 1 << 28))
        hi = lo + (width if b % 4 else int(rng.integers(0, width)))
        parts = [contribution(rng, lo, hi, int(rng.integers(0, 6))) for _ in range(P)]
        if b % 5:
            parts[P // 2] = picks(rng, lo, hi, 20_000)
        regions.append((lo, hi, parts))
    run_batch(regions, P, width, int(share * width), lead=lead)
