"""The slim tiles of the reduce (floats for a slot's first entry, a list for the others) at
the edges of what they hold: hit slots, listed entries and units up to and one past the limit,
slots that many contributions share, both kinds of bitmap, room for more outputs than the last-level
cache holds.

Sums are of dyadic values small enough that fp64 adds them exactly in any order, so the oracle's
result is the only correct one, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2201_07598_amd as okt
from test_gpu_reduce_tiles import DEV, dev, run_batch

pytestmark = pytest.mark.gpu
HITS, LIST = 6912, 2968


def tile(rng, lo, span, P, distinct, again, most=1 << 30):
    """P contributions that hit `distinct` of the first `span` slots from lo, with `again` entries more
    than that: each slot hit by at most `most`."""
    slots = np.sort(rng.choice(span, distinct, replace=False))
    owner = rng.permutation(np.arange(distinct) % P)             # all as long as each other
    have = [set(slots[owner == p].tolist()) for p in range(P)]
    hot = slots[: max(1, -(-again // max(1, min(most, P) - 1)))]      # slots that take the rest
    left = again
    for s in hot.tolist():
        for p in range(P):
            if left and s not in have[p]:
                have[p].add(s)
                left -= 1
    assert left == 0
    return [(np.array(sorted(h), dtype=np.int64) + lo).astype(np.uint32) for h in have]


def regions_of(make, B, P, width):
    """B regions with one entry a contribution, and `make`'s at both ends of the launch."""
    los = [b * 1_013 for b in range(B)]
    return [(lo, lo + width, make(lo) if lo in (0, los[-1]) else [np.array([lo + 3 * p], np.uint32) for p in range(P)])
            for lo in los]


# P, distinct, again, most
LONG_CASES = [
    (40, HITS, 0, 2), (40, HITS + 1, 0, 2), (40, HITS, 1, 2), (40, 1, 39, 40),
    (40, 4000, LIST, 2), (40, 4000, LIST + 1, 2), (40, 4000, LIST, 40), (40, 5000, 1536, 3), (40, 5000, 1537, 40),
    (64, 8192 - 64, 0, 2), (64, 6000, 2192, 64), (64, 6000, 2193, 64), (128, 512, 2900, 128), (127, 511, 511, 2),
    (33, 6000, 500, 33)]
LONG_B, LONG_WIDTH, LONG_CAPACITIES = 52, 1_000_001, (33_000, 5_000)


@pytest.mark.parametrize("P,distinct,again,most", LONG_CASES)
def test_what_a_tile_holds(P, distinct, again, most):
    """Tiles of 98,304 slots, planned for few hits; the hits lie in the first of a region."""
    rng = np.random.default_rng(P * 7 + distinct + again)
    regions = regions_of(lambda lo: tile(rng, lo, 39_000, P, distinct, again, most), LONG_B, P, LONG_WIDTH)
    for capacity in LONG_CAPACITIES:                              # the second cuts outputs short
        run_batch(regions, P, LONG_WIDTH, capacity, lead=P % 4)


FULL_CASES = [(16, HITS, 0, 2), (16, HITS + 1, 0, 2), (16, 4000, LIST, 2), (16, 4000, LIST + 1, 16), (16, 6000, 2192, 16),
              (16, 6000, 2193, 16), (32, HITS, 1, 2), (32, 5000, 2500, 32)]
FULL_B, FULL_WIDTH, FULL_CAPACITY = 24, 1_300_001, 195_000


@pytest.mark.parametrize("P,distinct,again,most", FULL_CASES)
def test_what_a_full_tile_holds(P, distinct, again, most):
    """Tiles of up to 65,536 slots that are planned for as many hits as they hold."""
    rng = np.random.default_rng(P * 7 + distinct + again)
    regions = regions_of(lambda lo: tile(rng, lo, 39_000, P, distinct, again, most), FULL_B, P, FULL_WIDTH)
    run_batch(regions, P, FULL_WIDTH, FULL_CAPACITY, lead=P % 4)


# P, width, span, distinct, again, capacity
KIND_CASES = [
    (70, 98_304, 98_304, 5_000, 700, 5_900), (70, 65_536 * 9, 65_536, 6_000, 1_000, 35_000),
    (3, 3_000_001, 40_000, 3_000, 2_500, 130_000), (7, 2_000_001, 40_000, 3_000, 2_500, 240_000),
    (8, 2_000_001, 40_000, 5_000, 1_000, 240_000), (64, 60_001, 60_001, 5_000, 900, 6_000), (40, 60_001, 60_001, 2_500, 400, 2_900),
    # 530 x 64,000 entries of eight bytes: more than the last-level cache
    (70, 1_600_001, 150_000, 9_000, 900, 64_000)]


def kind_batch(width):
    return 40 if width > 1_999_999 else 530


@pytest.mark.parametrize("P,width,span,distinct,again,capacity", KIND_CASES)
def test_kinds_of_slim_tiles(P, width, span, distinct, again, capacity):
    """Wide bitmaps and the widest, few contributions in long regions, room for many outputs."""
    rng = np.random.default_rng(width + distinct)
    regions = regions_of(lambda lo: tile(rng, lo, span, P, distinct, again), kind_batch(width), P, width)
    run_batch(regions, P, width, capacity, lead=1)


# P, distinct, again: tiles that go by windows of at most 3,568 hits (98,304 slots each).
# One window of more entries than registers hold, read by chunks and streamed; several, their slices'
# ends found at once (36 contributions) and in turn (P * windows > 1,024); more than 16 bits count
WINDOW_CASES = [(40, 3_000, 9_000), (40, 3_500, 20_000), (36, 20_000, 3_000), (36, 98_304, 0), (40, 98_304, 300),
                (64, 70_000, 9_000), (128, 30_000, 6_000), (128, 98_304, 0), (20, 4_500, 12_000), (7, 98_304, 2_000)]
WINDOW_B, WINDOW_WIDTH, WINDOW_CAPACITY = 12, 5_000_001, 120_000


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("P,distinct,again", WINDOW_CASES)
def test_windows_of_slim_tiles(P, distinct, again, dense):
    rng = np.random.default_rng(P + distinct)
    regions = regions_of(lambda lo: tile(rng, lo, 98_304, P, distinct, again), WINDOW_B, P, WINDOW_WIDTH)
    run_batch(regions, P, WINDOW_WIDTH, WINDOW_CAPACITY, lead=P % 4, dense=dense)


VALUES_CALL, VALUES_CAPACITY = (40, 40_003, 520), 1_900


def test_values_that_are_no_ordinary_numbers():
    """A lone -0 leaves as +0, as an fp64 sum that starts at +0 makes of it; NaN, infinities and
    subnormals stay what they are, alone and in sums."""
    P, width, B = VALUES_CALL
    special = np.array([-0.0, np.nan, np.inf, -np.inf, 1e-45, -1e-45, 0.0, 3.0e38], np.float32)
    first = np.arange(0, 16, dtype=np.uint32)                    # contribution 0: each value twice
    second = np.arange(8, 16, dtype=np.uint32)                   # contribution 1: the second eight once more
    idx = np.concatenate([np.concatenate([first, second]) + np.uint32(7 * b) for b in range(B)])
    val = np.tile(np.concatenate([special, special, special]), B)
    off = np.zeros((B, P + 1), np.uint64)
    off[:, 0] = 24 * np.arange(B)
    off[:, 1] = off[:, 0] + 16
    off[:, 2:] = (off[:, 0] + 24)[:, None]
    lo_hi = np.stack([7 * np.arange(B), 7 * np.arange(B) + width], 1).astype(np.uint32)
    cap = VALUES_CAPACITY
    o_idx = torch.zeros(B * cap, dtype=torch.int32, device=DEV)
    o_val = torch.zeros(B * cap, device=DEV)
    nnz = torch.zeros(2 * B, dtype=torch.int64, device=DEV)
    ws = torch.empty(okt.okt_sparse_reduce_batch_workspace_bytes(B, P, width), dtype=torch.uint8, device=DEV)
    okt.okt_sparse_reduce_batch(dev(idx), dev(val), dev(off.reshape(-1)), dev(lo_hi.reshape(-1)), B, P, width, o_idx,
                                o_val, cap, nnz, ws)
    torch.cuda.synchronize()
    assert (nnz == 16).all()
    with np.errstate(over="ignore", invalid="ignore"):
        want = np.concatenate([0.0 + special.astype(np.float64), special.astype(np.float64) * 2]).astype(np.float32)
    got = o_val.cpu().numpy().reshape(B, cap)[:, :16]
    assert np.array_equal(got, np.broadcast_to(want, got.shape), equal_nan=True)
    assert np.array_equal(np.signbit(got[:, [0, 6, 8, 14]]), np.zeros((B, 4), bool))


REPLAY_CALL = (64, 60_001, 520, 6_000)


def test_dense_copy_and_replays():
    """The dense regions beside the sparse outputs, eager and from a captured graph replayed on other
    values, with another launch in the workspace in between."""
    rng = np.random.default_rng(5)
    P, width, B, cap = REPLAY_CALL
    ps = tile(rng, 0, 39_000, P, 5_000, 1_200)
    one = np.concatenate(ps)
    idx = np.concatenate([one, np.concatenate([np.array([3 * p], np.uint32) for p in range(P)])])
    off = np.zeros((B, P + 1), np.uint64)
    off[0] = np.concatenate([[0], np.cumsum([p.size for p in ps])])
    off[1:] = one.size + np.arange(P + 1)                        # all others share one short input
    lo_hi = np.tile(np.array([0, width], np.uint32), B)
    d_idx, d_off, d_lo_hi = dev(idx), dev(off.reshape(-1)), dev(lo_hi)
    vals = [(rng.integers(-2048, 2048, idx.size) * 2.0 ** -12).astype(np.float32) for _ in range(2)]
    d_val = dev(vals[0]).clone()
    o_idx = torch.zeros(B * cap, dtype=torch.int32, device=DEV)
    o_val = torch.zeros(B * cap, device=DEV)
    dense = torch.full((B * width,), 7.0, device=DEV)
    nnz = torch.zeros(2 * B, dtype=torch.int64, device=DEV)
    ws = torch.empty(okt.okt_sparse_reduce_batch_workspace_bytes(B, P, width), dtype=torch.uint8, device=DEV)

    def call():
        okt.okt_sparse_reduce_batch(d_idx, d_val, d_off, d_lo_hi, B, P, width, o_idx, o_val, cap, nnz, ws, dense_out=dense)

    def check(val):
        torch.cuda.synchronize()
        for b, part in ((0, slice(0, one.size)), (1, slice(one.size, None)), (B - 1, slice(one.size, None))):
            full = np.zeros(width)
            np.add.at(full, idx[part], val[part].astype(np.float64))
            hit = np.unique(idx[part])
            assert nnz[2 * b:2 * b + 2].tolist() == [hit.size, hit.size]
            assert np.array_equal(o_idx[b * cap:b * cap + hit.size].cpu().numpy().view(np.uint32), hit)
            assert np.array_equal(o_val[b * cap:b * cap + hit.size].cpu().numpy(), full[hit].astype(np.float32))
            assert np.array_equal(dense[b * width:(b + 1) * width].cpu().numpy(), full.astype(np.float32))

    call()
    check(vals[0])
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        call()
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            call()
    for i in range(4):
        d_val.copy_(dev(vals[i % 2]))
        dense.fill_(7.0), o_val.zero_(), nnz.zero_()
        graph.replay()
        check(vals[i % 2])
        ws.random_(0, 255)                                       # garbage between the replays
