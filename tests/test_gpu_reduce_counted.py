"""Regions of many narrow tiles whose launch counts the hit slots of every tile first:
around the number of tiles from which it does, with every number of lanes that search a
slice's end, dense, ranked and sparse tiles, and parts of the region that are hit far
more than planned.  Sums are of dyadic values, so the oracle's result is the only
correct one, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2201_07598_amd as okt
from oracle import okt_oracle as orc
from tests.okt_harness import DEV, to_dev, u32, u64

pytestmark = pytest.mark.gpu


def check(parts, lo, hi, capacity, lead=0, dense=True):
    P = len(parts)
    off = np.concatenate([[0], np.cumsum([p.size for p in parts])]).astype(np.uint64)
    idx = np.concatenate(parts).astype(np.uint32)
    val = (np.random.default_rng(idx.size).integers(-2048, 2048, idx.size) * 2.0 ** -12).astype(np.float32)
    # `lead` words in front: slices start at every word address; the input ends with the buffer
    d_idx = to_dev(np.concatenate([np.zeros(lead, np.uint32), idx]))[lead:]
    d_val = to_dev(np.concatenate([np.zeros(lead, np.float32), val]))[lead:]
    out_idx = torch.full((max(capacity, 1),), -1, dtype=torch.int32, device=DEV)
    out_val = torch.zeros(max(capacity, 1), device=DEV)
    nnz = torch.zeros(2, dtype=torch.int64, device=DEV)
    d_dense = torch.full((hi - lo,), 7.0, device=DEV) if dense else None
    ws = torch.full((okt.okt_workspace_bytes(hi - lo, P),), 0xA5, dtype=torch.uint8, device=DEV)
    okt.okt_sparse_reduce(d_idx, d_val, to_dev(off), lo, hi, out_idx, out_val, nnz, ws, dense_out=d_dense,
                          capacity=capacity)
    ref = orc.sparse_reduce(idx, val, off, lo, hi)
    total = ref["idx"].size
    emitted = min(total, capacity)
    assert tuple(int(x) for x in u64(nnz)) == (emitted, total)
    assert np.array_equal(u32(out_idx[:emitted]), ref["idx"][:emitted])
    assert np.array_equal(out_val[:emitted].cpu().numpy(), ref["val"][:emitted].astype(np.float32))
    assert bool((out_idx[emitted:] == -1).all())
    if dense:
        assert np.array_equal(d_dense.cpu().numpy(), ref["dense"].astype(np.float32))


def picks(rng, lo, width, m):
    return (np.sort(rng.choice(width, min(m, width), replace=False)) + lo).astype(np.uint32)


# narrow dense tiles are 4096 slots: 127 of them take tickets, 128 do not (up to 96 contributions)
@pytest.mark.parametrize("width", [127 * 4096, 127 * 4096 + 1, 128 * 4096 + 5, 700_001])
@pytest.mark.parametrize("P", [1, 2, 16, 17, 33, 96, 97, 100, 256, 257])
def test_dense_tiles(width, P):
    rng = np.random.default_rng(width + P)
    lo = 3_000_001
    parts = [picks(rng, lo, width, int(rng.integers(0, 2 * width // P))) for _ in range(P)]
    check(parts, lo, lo + width, width, lead=P % 4)


@pytest.mark.parametrize("P,m,width", [(1, 300_000, 3_000_000), (3, 200_000, 3_400_000), (32, 34_375, 3_437_500),
                                       (33, 4_000, 4_000_000), (96, 1_500, 6_400_000), (200, 700, 6_400_000), (256, 2_000, 3_500_000)])
def test_ranked_and_sparse_tiles(P, m, width):
    rng = np.random.default_rng(P)
    lo = 17
    parts = [picks(rng, lo, width, m) for _ in range(P)]
    if P > 2:                                            # (without any entry there would be no buffer)
        parts[0] = np.zeros(0, np.uint32)
        parts[1] = np.array([lo, lo + width - 1], np.uint32)
        parts[2] = picks(rng, lo, 5_000, 4_000)          # all of it in the first tile
    union = np.unique(np.concatenate(parts)).size
    check(parts, lo, lo + width, union, lead=1)
    check(parts, lo, lo + width, union // 2, dense=False)


def test_entries_far_from_where_they_were_planned():
    """Most entries in a tenth of the region: tiles with more entries than registers hold
    and more hit slots than accumulators, next to empty ones; guesses that miss."""
    rng = np.random.default_rng(9)
    lo, width, P = 1_000, 3_000_000, 24
    parts = [np.unique(np.concatenate([picks(rng, lo + width // 2, width // 10, 40_000), picks(rng, lo, width, 500)]))
             for _ in range(P)]
    check(parts, lo, lo + width, P * 40_500)


def test_the_end_of_the_index_space():
    rng = np.random.default_rng(10)
    hi, width = (1 << 32) - 1, 900_000
    parts = [np.unique(np.concatenate([picks(rng, hi - width, width, 60_000), np.array([hi - 1], np.uint32)]))
             for _ in range(8)]
    check(parts, hi - width, hi, 480_100)
