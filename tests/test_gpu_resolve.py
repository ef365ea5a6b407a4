"""The exact threshold and the refresh iteration where their launches, shares and
digits change: vector lengths around the limits of each form, candidates that fill
one share of a workgroup or just more, answers far above the sample's bound, bounds
above the answer, ties.  Everything against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2201_07598_amd as okt
from oracle import okt_oracle as orc
from tests import sample_replay as sr
from tests.okt_harness import DEV, bits_equal, to_dev, u32, u64, workspace
from tests.test_gpu_refresh import check_refresh, lap

pytestmark = pytest.mark.gpu


def check_threshold(acc, k, ws_bytes=None):
    th = torch.full((1,), -7.0, device=DEV)
    cnt = torch.zeros(1, dtype=torch.int64, device=DEV)
    ws = workspace(okt.okt_workspace_bytes(acc.size, 0) if ws_bytes is None else ws_bytes)
    ws.fill_(0xAB)
    okt.okt_topk_threshold_exact(to_dev(acc), k, th, cnt, ws)
    torch.cuda.synchronize()
    rth, rcnt = orc.topk_threshold_exact(acc, k, method="sort" if acc.size < 5000 else "partition")
    assert th.cpu().numpy().view(np.uint32)[0] == np.float32(rth).view(np.uint32)
    assert int(u64(cnt)[0]) == rcnt


@pytest.mark.parametrize("n", [1, 2, 4097, 16_383, 16_384, 16_385, 32_768, 32_769, 65_536, 65_537, 70_001,
                               131_071, 131_072, 131_073, 300_007, 2_097_152, 2_097_153, 2_200_003])
def test_threshold_lengths(n):
    acc = lap(n, n)
    acc[n // 2::7] = 0.0
    for k in sorted({1, max(1, n // 1000), max(1, n // 50), max(1, n // 3), n}):
        check_threshold(acc, k)
    check_threshold(acc, max(1, n // 50), ws_bytes=64 * 1024)
    same = np.full(n, -0.5, dtype=np.float32)
    check_threshold(same, max(1, n // 50))
    check_threshold(np.zeros(n, np.float32), max(1, n // 50))


# k and the candidates it brings (about 1.3 k): one row, several, around 24,576, many shares
@pytest.mark.parametrize("n,k", [(131_072, 40), (300_007, 3_000), (1_000_003, 17_500), (1_000_003, 18_500),
                                 (1_000_003, 20_500), (3_000_001, 60_000), (5_000_011, 300_000),
                                 (5_000_011, 400_000)])
def test_refresh_shares_of_candidates(n, k):
    g, e = lap(n + k, n), lap(n + k + 1, n, 2e-3)
    check_refresh(g, e, 0.25, k, 2 * k)
    check_refresh(g, e, 0.25, k, k // 2 + 1)


def with_candidates(acc, k, count):
    """`acc` changed where the sample does not look, so that exactly `count` elements pass
    its bound for k."""
    bound = sr.bounds_dense(acc, k).min()
    passing, free = sr.key_of(acc) >= bound, ~sr.sampled(acc.size)
    there = int(passing.sum())
    if there > count:
        acc[np.flatnonzero(passing & free)[:there - count]] = 0.0
    else:
        low = np.flatnonzero(~passing & free)[:count - there]
        acc[low] = np.array([bound], np.uint32).view(np.float32)[0] * np.linspace(1.0, 1.5, low.size, dtype=np.float32)
    assert sr.bounds_dense(acc, k).min() == bound
    assert np.count_nonzero(sr.key_of(acc) >= bound) == count
    return acc


# The candidates' limits: a single share of the threshold alone and one of the refresh that
# takes no vote on it (24,576), the rows after that, the largest single share (40,960).
# Spread keys are a single share there, keys that are alike are several.
@pytest.mark.parametrize("count", [24_575, 24_576, 24_577, 28_673, 32_769, 36_864, 36_865, 40_959, 40_960, 40_961])
@pytest.mark.parametrize("values", [0, 1, 3])
def test_candidates_at_the_limits_of_a_single_share(count, values):
    n, k = 1_000_003, int(count / 1.28)
    g = lap(count + values, n)
    if values:
        top = np.argpartition(-np.abs(g), 2 * k)[:2 * k]
        g[top] = np.random.default_rng(count).choice(np.array([0.25, -0.375, 0.5][:values], np.float32), 2 * k)
        k = 2 * k * 9 // 16 if values == 3 else k                  # among the two larger of the three; a tie
    g = with_candidates(g, k, count)
    check_threshold(g, k)
    for cap in (count, k, k // 3):
        check_refresh(g, np.zeros(n, np.float32), 1.0, k, cap)


@pytest.mark.parametrize("n", [200_003, 2_500_003, 4_300_003])
def test_answers_far_from_the_bound(n):
    rng = np.random.default_rng(n)
    k = n // 100
    zero = np.zeros(n, np.float32)
    # exactly k large values over a floor of small ones: the bound lies among the small,
    # the answer octaves above it
    g = lap(7, n, 1e-6)
    at = rng.choice(n, k, replace=False)
    g[at] = rng.choice([-1.0, 1.0], k) * rng.uniform(1.0, 2.0, k)
    for kk in (k, k - 1, k // 2):
        check_refresh(g, zero, 1.0, kk, 2 * k)
        check_threshold(g, kk)
    # a handful of values, most of the vector tied at the answer or just below it
    t = rng.choice(np.array([0.0, 1e-3, -1e-3, 3e-3], np.float32), n, p=[0.5, 0.2, 0.2, 0.1]).astype(np.float32)
    for kk in (k, n // 10, n // 10 + 5, n // 3):
        check_refresh(t, zero, 1.0, kk, n)
        check_threshold(t, kk)
    # values over the whole range of exponents, a NaN and infinities on top
    w = (2.0 ** rng.uniform(-140, 120, n)).astype(np.float32) * rng.choice([-1, 1], n).astype(np.float32)
    w[5], w[6], w[n - 1] = np.nan, np.inf, -np.inf
    for kk in (1, 2, 3, 4, k):
        check_refresh(w, zero, 1.0, kk, 2 * k)
        check_threshold(w, kk)


@pytest.mark.parametrize("n", [1_000_003, 4_300_003])
def test_a_sample_that_sees_only_large_values(n):
    """Every run of sixteen that the sample reads is large, everything else small:
    each bound lies above the answer, too few candidates are found, and the whole
    vector decides."""
    g = lap(9, n, 1e-6)
    seen = sr.sampled(n)
    g[seen] = lap(n, int(seen.sum()), 1.0) + np.float32(2.0)
    k = 150_000 if n < 2_000_000 else 300_000
    for kk in (k, n // 13):
        assert np.count_nonzero(sr.key_of(g) >= sr.bounds_dense(g, kk).min()) < kk
        check_refresh(g, np.zeros(n, np.float32), 1.0, kk, 2 * kk)
        check_threshold(g, kk)


# lengths around a step of the streaming digit passes (4096 elements), around the point
# where their workgroups take a second step (two per compute unit), and from which they
# read around the cache
@pytest.mark.parametrize("n", [2_097_153, 2_097_152 + 4_096, 2_097_152 + 4_097, 2 * 2_097_152 - 1,
                               6_291_459, 67_108_864, 67_108_867])
def test_digit_passes_over_the_whole_vector(n):
    acc = lap(n, n)
    acc[n // 3:n // 3 + 200_000] = 0.0
    acc[n - 1], acc[n - 2] = np.inf, np.nan
    acc[5_000:5_300] = np.float32(-2.5e-3)
    above = int((np.abs(acc) > np.float32(2.5e-3)).sum()) + 1              # and the NaN
    for k in (above + 150, n // 2) if n > 10_000_000 else (1, 2, 3, above + 1, above + 300, n // 3, n):
        check_threshold(acc, k, ws_bytes=64 * 1024)
    if n < 10_000_000:
        check_threshold(np.zeros(n, np.float32), n // 100, ws_bytes=64 * 1024)
        check_threshold(np.full(n, -0.5, np.float32), n, ws_bytes=64 * 1024)


@pytest.mark.parametrize("n,k", [(100_003, 4_000), (300_007, 9_000), (2_500_003, 60_000)])
@pytest.mark.parametrize("tied", [15, 16, 17, 40, 63, 64])
def test_candidates_that_share_a_bin(n, k, tied):
    """Of every 64 large values `tied` are equal (CROWD of a wave's lanes, just fewer and
    more, all of them): one add counts those, and no element is counted twice or lost.
    Candidates that fit one share, and many."""
    rng = np.random.default_rng(n + tied)
    g = lap(n, n, 1e-6)
    large = int(1.5 * k)
    at = np.sort(rng.choice(n, large, replace=False))
    value = rng.uniform(1.0, 1.9, large).astype(np.float32)
    value[np.arange(large) % 64 < tied] = np.float32(1.5)
    g[at] = value * rng.choice(np.array([-1.0, 1.0], np.float32), large)
    above = int((value > np.float32(1.5)).sum())
    for kk in sorted({above + 1, above + 7, k, large - 1} | ({above} if above else set())):
        check_threshold(g, kk)
        check_refresh(g, np.zeros(n, np.float32), 1.0, kk, large)
    check_threshold(g, k, ws_bytes=64 * 1024)


# candidates in one share and in many, vectors that one workgroup takes; up to 16 keys are
# ranked instead of counted
@pytest.mark.parametrize("n,k", [(4_003, 40), (60_001, 600), (300_007, 3_000), (2_500_003, 60_000)])
@pytest.mark.parametrize("close", [1, 2, 15, 16, 17, 63, 64, 65])
def test_the_last_digit_of_a_few_keys(n, k, close):
    """`close` keys that differ in the lowest bits alone, some of them equal, and the answer
    among them: the first, one in the middle, the last, and its neighbours on both sides."""
    rng = np.random.default_rng(n + close)
    g = lap(n, n, 1e-6)
    large = max(int(1.3 * k), 4 * close)
    bits = np.float32(1.25).view(np.uint32) + rng.choice(400, close, replace=False).astype(np.uint32)
    bits[close // 2:close // 2 + 2] = bits[close // 2]
    value = rng.uniform(1.0, 1.9, large).astype(np.float32)
    value[(value > 1.24) & (value < 1.26)] = np.float32(1.3)
    value[rng.choice(large, close, replace=False)] = bits.view(np.float32)
    at = rng.choice(n, large, replace=False)
    g[at] = value * rng.choice(np.array([-1.0, 1.0], np.float32), large)
    above = int((value > 1.28).sum())
    for kk in (above, above + 1, above + (close + 1) // 2, above + close, above + close + 1):
        check_threshold(g, kk)
        check_refresh(g, np.zeros(n, np.float32), 1.0, kk, large)


@pytest.mark.parametrize("n", [70_001, 300_007, 2_500_003, 4_300_003])
def test_a_sample_that_sees_zeros(n):
    """Fewer than k elements that are not zero: the sample's bound is zero.  The answer is
    zero, or, where just enough elements are not, the least of them: a subnormal, which
    the digits from zero up find, or a value far above, which they do not."""
    k = n // 100
    rng = np.random.default_rng(n)
    for nonzero, low in ((0, 1.0), (k // 10, 1.0), (k - 1, 1.0), (k, 1.0), (k, 1e-41), (k + 3, 1e-38)):
        g = np.zeros(n, np.float32)
        at = rng.choice(n, nonzero, replace=False)
        g[at] = (low * rng.uniform(1.0, 1.9, nonzero)).astype(np.float32) * rng.choice(
            np.array([-1.0, 1.0], np.float32), nonzero)
        check_threshold(g, k)
        check_refresh(g, np.zeros(n, np.float32), 1.0, k, n if nonzero < k else k + 10)


@pytest.mark.parametrize("n,k", [(300_007, 3_000), (2_000_003, 120_000), (4_300_003, 120_000)])
def test_digit_waits_that_give_up_are_reported(n, k):
    """With the waits between the digits limited to one poll a call completes or reports
    UINT64_MAX counts; it never hangs.  Candidates in one share (no wait at all), digits
    over a vector with a bound, candidates in many shares with the select behind."""
    g, e = lap(n + 9, n), lap(n + 10, n, 2e-3)
    acc = orc.residual_accumulate(g, e, 0.5)
    rth, rcnt = orc.topk_threshold_exact(acc, k, method="partition")
    ridx, rval, rres, total = orc.threshold_select(acc, rth, capacity=2 * k)
    bad = 0xFFFFFFFFFFFFFFFF
    th = torch.zeros(1, device=DEV)
    cnt = torch.zeros(1, dtype=torch.int64, device=DEV)
    idx = torch.full((2 * k,), -1, dtype=torch.int32, device=DEV)
    val = torch.zeros(2 * k, device=DEV)
    nnz = torch.zeros(2, dtype=torch.int64, device=DEV)
    ws = workspace(okt.okt_workspace_bytes(n, 0))
    d_acc, d_g = to_dev(acc), to_dev(g)
    outcomes = []
    okt.okt_debug_digit_spin_limit(1)
    try:
        for _ in range(3):
            cnt.fill_(-5)
            okt.okt_topk_threshold_exact(d_acc, k, th, cnt, ws)
            torch.cuda.synchronize()
            c = int(u64(cnt)[0])
            outcomes.append(c == bad)
            if c != bad:
                assert c == rcnt and th.cpu().numpy().view(np.uint32)[0] == np.float32(rth).view(np.uint32)
            cnt.fill_(-5), nnz.fill_(-5)
            d_e = to_dev(e)
            okt.okt_accumulate_topk_select(d_g, d_e, 0.5, k, th, cnt, idx, val, nnz, ws)
            torch.cuda.synchronize()
            c, m = int(u64(cnt)[0]), [int(x) for x in u64(nnz)]
            outcomes.append(m[1] == bad)
            if bad in m:
                assert m == [bad, bad] and c in (bad, rcnt)
            else:
                assert c == rcnt and m == [ridx.size, total]
                assert np.array_equal(u32(idx[:total]), ridx) and bits_equal(d_e.cpu().numpy(), rres)
    finally:
        okt.okt_debug_digit_spin_limit(0)
    print(outcomes, flush=True)
    check_threshold(acc, k)                          # the limit restored: exact again
    check_refresh(g, e, 0.5, k, 2 * k)


@pytest.mark.parametrize("n", [70_001, 131_073, 300_007, 2_500_003, 5_000_011])
def test_the_sample_is_the_one_the_host_replays(n):
    """The bounds that the sample leaves in the workspace, and how many candidates the
    collection finds with the least of them: what the tests that mislead the sample, or
    count on it, take for granted."""
    g, e = lap(n + 1, n), lap(n + 2, n, 2e-3)
    acc = orc.residual_accumulate(g, e, 0.5)
    th = torch.zeros(1, device=DEV)
    cnt = torch.zeros(1, dtype=torch.int64, device=DEV)
    ws = workspace(okt.okt_workspace_bytes(n, 0))
    for k in (1, n // 1000, n // 50):
        bounds = sr.bounds_dense(acc, k)
        passing = int(np.count_nonzero(sr.key_of(acc) >= bounds.min()))
        assert k <= passing <= n // 8              # the room that okt_workspace_bytes gives
        okt.okt_topk_threshold_exact(to_dev(acc), k, th, cnt, ws)
        state = sr.State(ws)
        assert np.array_equal(state.bounds, bounds) and state.keys_found == passing
        if n >= 131_072:
            idx = torch.zeros(2 * k, dtype=torch.int32, device=DEV)
            val = torch.zeros(2 * k, device=DEV)
            nnz = torch.zeros(2, dtype=torch.int64, device=DEV)
            okt.okt_accumulate_topk_select(to_dev(g), to_dev(e), 0.5, k, th, cnt, idx, val, nnz, ws)
            state = sr.State(ws)
            assert np.array_equal(state.bounds, bounds) and state.collected == passing
