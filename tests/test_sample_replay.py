"""The host replay of the threshold's sample against the kernel's source and against a
sample taken literally."""
import os
import re

import numpy as np
import pytest

from tests import sample_replay as sr

SOURCE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                      "paper_2201_07598_amd", "csrc", "okt_threshold.hip")


def test_the_replay_has_the_kernels_geometry():
    text = open(SOURCE).read()
    assert int(re.search(r"SAMPLE_RUN = (\d+)", text).group(1)) == sr.RUN
    assert int(re.search(r"SAMPLE_RUNS = (\d+)", text).group(1)) == sr.RUNS
    assert int(re.search(r"constexpr int BOUNDS = (\d+)", text).group(1)) == sr.WORKGROUPS
    m = re.search(r"SAMPLE_SHIFT = (\d+) - (\d+)", text)
    assert int(m.group(1)) - int(m.group(2)) == sr.SHIFT


@pytest.mark.parametrize("n", [65_537, 131_072, 300_007, 5_000_011])
def test_the_replay_is_a_sample_taken_literally(n):
    rng = np.random.default_rng(n)
    acc = rng.laplace(0, 1e-3, n).astype(np.float32)
    acc[rng.random(n) < 0.5] = 0.0
    for k in (1, n // 1000, n // 50, n // 3, n):
        per_wg = sr.RUNS // sr.WORKGROUPS * sr.RUN
        kp = (k * per_wg + n // 2) // n
        rank = min(max(kp + int(np.sqrt(np.float32(kp)) + np.float32(0.5)), 1), per_wg)
        want = []
        for wg in range(sr.WORKGROUPS):
            runs = [int(r) * (n // sr.RUN) // sr.RUNS for r in range(wg, sr.RUNS, sr.WORKGROUPS)]
            keys = np.concatenate([sr.key_of(acc[16 * r:16 * r + 16]) for r in runs])
            want.append(int(np.sort(keys)[::-1][rank - 1]) >> sr.SHIFT << sr.SHIFT)
        assert np.array_equal(sr.bounds_dense(acc, k), np.array(want, np.uint32)), k


def test_positions_at_the_longest_length():
    n = (1 << 32) - 1
    starts = sr.run_starts(n)
    assert int(starts[-1]) == 8191 * (n // 16) // 8192 * 16 and int(starts[-1]) + 16 <= n
    pos = starts[[0, 1, 17, 8191]].astype(np.int64) + 3
    b = sr.bounds(n, 500, pos, sr.key_of(np.array([1.0, 2.0, 0.5, 4.0], np.float32)))
    assert np.count_nonzero(b) == 3 and int(b[1]) == int(sr.key_of(np.array([2.0]))[0])
