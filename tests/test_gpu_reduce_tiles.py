"""The reduce's tiles where they can go wrong: the wide form (a launch with enough
regions to fill the chip), contribution counts around the number of threads, units
that end a slice, a contribution or the input, tiles with more entries than
registers hold, more hit slots than accumulators, and more than 16 bits count.

Sums are of dyadic values small enough that fp64 adds them exactly in any order, so
the oracle's result is the only correct one, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2201_07598_amd as okt
from oracle import okt_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a):
    view = {np.dtype(np.uint32): np.int32, np.dtype(np.uint64): np.int64}.get(a.dtype)
    return torch.from_numpy(np.ascontiguousarray(a).view(view) if view else a).to(DEV)


def run_batch(regions, P, width, capacity, lead=0, ws_share=1.0, dense=False):
    """regions: list of (lo, hi, [P index arrays]); checks every region against the oracle."""
    B = len(regions)
    parts = [p for _, _, ps in regions for p in ps]
    lens = np.array([p.size for p in parts], dtype=np.int64).reshape(B, P)
    idx = np.concatenate(parts + [np.zeros(0, np.uint32)]).astype(np.uint32)
    rng = np.random.default_rng(idx.size + P)
    val = (rng.integers(-2048, 2048, idx.size) * 2.0 ** -12).astype(np.float32)
    off = np.zeros((B, P + 1), dtype=np.uint64)
    starts = np.concatenate([[0], np.cumsum(lens.reshape(-1))]).astype(np.uint64)
    for b in range(B):
        off[b] = starts[b * P:b * P + P + 1]
    # `lead` words in front: slices start at every word address, the input ends with the buffer
    d_idx = torch.zeros(lead + idx.size, dtype=torch.int32, device=DEV)[lead:]
    d_val = torch.zeros(lead + idx.size, device=DEV)[lead:]
    d_idx.copy_(dev(idx)), d_val.copy_(dev(val))
    lo_hi = dev(np.array([(a, b) for a, b, _ in regions], dtype=np.uint32).reshape(-1))
    o_idx = torch.full((B * max(capacity, 1),), -1, dtype=torch.int32, device=DEV)
    o_val = torch.zeros(B * max(capacity, 1), device=DEV)
    nnz = torch.zeros(2 * B, dtype=torch.int64, device=DEV)
    told = okt.okt_sparse_reduce_batch_workspace_bytes(B, P, width)
    ws = torch.empty(int(ws_share * told), dtype=torch.uint8, device=DEV)
    d_dense = torch.full((B * width,), 7.0, device=DEV) if dense else None
    okt.okt_sparse_reduce_batch(d_idx, d_val, dev(off.reshape(-1)), lo_hi, B, P, width, o_idx, o_val,
                                capacity, nnz, ws, dense_out=d_dense)
    torch.cuda.synchronize()
    got_i, got_v = o_idx.cpu().numpy().view(np.uint32), o_val.cpu().numpy()
    nnz = nnz.cpu().numpy().reshape(B, 2)
    for b, (lo, hi, _) in enumerate(regions):
        s, e = int(off[b, 0]), int(off[b, P])
        ref = orc.sparse_reduce(idx[s:e], val[s:e], off[b] - off[b, 0], lo, hi)
        U = ref["idx"].size
        n = min(U, capacity)
        assert tuple(nnz[b]) == (n, U), (b, nnz[b], U)
        at = b * capacity
        assert np.array_equal(got_i[at:at + n], ref["idx"][:n]), b
        assert np.array_equal(got_v[at:at + n], ref["val"][:n].astype(np.float32)), b
        if dense:
            full = np.zeros(hi - lo, np.float32)
            full[ref["idx"].astype(np.int64) - lo] = ref["val"].astype(np.float32)
            assert np.array_equal(d_dense[b * width:b * width + hi - lo].cpu().numpy(), full), b


def some(rng, lo, width, m):
    return (np.sort(rng.choice(width, min(m, width), replace=False)) + lo).astype(np.uint32)


@pytest.mark.parametrize("P,m,share", [
    (1, 700, 0.05), (3, 333, 0.2), (16, 16, 0.1), (16, 17, 0.34), (16, 95, 0.36), (64, 40, 0.05),
    (65, 3, 0.02), (256, 60, 0.3), (511, 5, 0.1), (512, 5, 0.1), (513, 5, 0.1), (700, 30, 0.9)])
def test_wide_tiles_in_batches(P, m, share):
    """At least two wide tiles to a compute unit.  `share`: what the capacity claims of
    the region is hit, which picks the kind of tile, right or wrong."""
    rng = np.random.default_rng(P * 1000 + m)
    width, B = 40_003, 530
    kinds = [some(rng, 0, width, m) for _ in range(P)]
    regions = []
    for b in range(B):
        lo = b * 7_919
        if b < 6:
            ps = [some(rng, lo, width, int(rng.integers(0, 2 * m))) for _ in range(P)]
        else:                                        # cheap for the host: one set, shifted
            ps = [kinds[(p + b) % P] + np.uint32(lo) for p in range(P)]
        regions.append((lo, lo + width - (b % 3) * 37, ps))
    check = [0, 1, 2, 3, 4, 5, 6, 7, B - 2, B - 1]
    keep = [r if i in check else (r[0], r[1], [p[:1] for p in r[2]]) for i, r in enumerate(regions)]
    run_batch(keep, P, width, int(share * width), lead=P % 4)


def test_wide_tiles_with_more_hits_than_they_have_room_for():
    """Estimated very sparse, in fact every slot hit, by one contribution and by three.  (So few
    contributions in so short regions take narrow tiles; wide and slim ones that are hit so are
    in test_gpu_reduce_wide.py and test_gpu_reduce_slim.py.)"""
    width, B, P = 98_304 + 1_000, 300, 3
    full = np.arange(width, dtype=np.uint32)
    none = np.zeros(0, np.uint32)
    regions = [(b * 10, b * 10 + width, [none, none, none]) for b in range(B)]
    regions[0] = (0, width, [full, none, none])
    regions[7] = (70, 70 + width, [full + np.uint32(70), full[::2] + np.uint32(70), full + np.uint32(70)])
    regions[B - 1] = (5, 5 + width, [none, none, full[5:]])
    run_batch(regions, P, width, 4_000)
    run_batch(regions, P, width, width // 20)


def clustered(rng, lo, width, blocks, per_block, length):
    """`per_block` indices in each of some stretches of `length` indices: hit far more than the rest."""
    parts = [some(rng, lo + int(at), length, per_block) for at in blocks]
    return np.unique(np.concatenate(parts)).astype(np.uint32)


@pytest.mark.parametrize("B,P,dense_part,share", [
    # one stretch that is hit throughout: 1 window and just over, 2, many
    (2, 1, 3_968, 0.05), (2, 1, 3_969, 0.05), (2, 3, 8_000, 0.05), (2, 8, 32_768, 0.05), (3, 40, 30_000, 0.02),
    (60, 33, 7_968, 0.02), (60, 33, 8_000, 0.02), (60, 48, 60_000, 0.02), (60, 64, 8_065, 0.02), (60, 100, 65_536, 0.02),
    # the ends of all windows of all slices do not fit in LDS: searched in turn
    (2, 300, 32_768, 0.02), (40, 512, 65_536, 0.02),
    # more contributions than threads: every window reads all entries
    (2, 513, 32_768, 0.02)])
def test_windows_of_a_tile(B, P, dense_part, share):
    """Tiles planned for a region hit evenly, with a stretch that is hit throughout: by
    one contribution, by several that share it, by pieces of all."""
    rng = np.random.default_rng(P + dense_part)
    width = 700_001
    regions = []
    for b in range(B):
        lo = b * 3_001
        whole = np.arange(dense_part, dtype=np.uint32) + np.uint32(lo + 100_000 + 17 * b)
        ps = [np.unique(np.concatenate([whole[p::max(1, P // 3)] if P > 1 else whole,
                                        some(rng, lo, width, 40)])).astype(np.uint32) for p in range(P)]
        regions.append((lo, lo + width, ps if b in (0, 1, B - 1) else [p[:2] for p in ps]))
    run_batch(regions, P, width, int(share * width) + B, lead=B % 4)
    run_batch(regions[:2], P, width, 5_000)                 # output cut short, inside a window
    run_batch(regions[:1], P, width, width)                 # planned for a densely hit region


@pytest.mark.parametrize("P,units", [(1, 256), (1, 257), (2, 300), (8, 512), (8, 513), (8, 700), (16, 256), (31, 400),
                                     (32, 1_100), (33, 640), (40, 641), (64, 512), (65, 513), (128, 1_400)])
@pytest.mark.parametrize("B", [1, 36])
def test_entries_beyond_a_chunk(B, P, units):
    """Contributions that hit the same slots: about `units` pieces of 16 entries to a tile,
    around one and two chunks of each form, and fewer hit slots than accumulators."""
    rng = np.random.default_rng(P * 31 + units)
    width = 900_001
    per = max(1, units // P) * 16
    regions = []
    for b in range(B):
        lo = 11 * b
        common = some(rng, lo, 30_000, min(3_900, per + 100))
        ps = [np.sort(rng.choice(common, min(per - (p % 3) * (per > 16), common.size), replace=False)).astype(np.uint32)
              for p in range(P)]
        regions.append((lo, lo + width, ps if b in (0, B - 1) else [p[:1] for p in ps]))
    run_batch(regions, P, width, 60_000 if B == 1 else 120_000, lead=P % 4)


@pytest.mark.parametrize("P", [1, 8, 32, 33, 64, 600])
def test_windows_with_the_dense_copy(P):
    """The dense region of a tile that is written in windows: every hit slot's sum, zeros elsewhere."""
    rng = np.random.default_rng(P)
    lo, width = 1_000, 300_007
    ps = [clustered(rng, lo, width, (0, 120_000, width - 9_000), max(1, 9_000 // P) if P > 1 else 9_000, 9_000)
          for _ in range(P)]
    ps[0] = np.unique(np.concatenate([ps[0], np.arange(lo + 120_000, lo + 129_000)])).astype(np.uint32)
    idx = np.concatenate(ps)
    val = (rng.integers(-2048, 2048, idx.size) * 2.0 ** -12).astype(np.float32)
    off = np.concatenate([[0], np.cumsum([p.size for p in ps])]).astype(np.uint64)
    ref = orc.sparse_reduce(idx, val, off, lo, lo + width)
    U = ref["idx"].size
    cap = U + 3
    o_idx = torch.zeros(cap, dtype=torch.int32, device=DEV)
    o_val, dense = torch.zeros(cap, device=DEV), torch.full((width,), 7.0, device=DEV)
    nnz = torch.zeros(2, dtype=torch.int64, device=DEV)
    ws = torch.empty(okt.okt_sparse_reduce_batch_workspace_bytes(1, P, width), dtype=torch.uint8, device=DEV)
    okt.okt_sparse_reduce(dev(idx), dev(val), dev(off), lo, lo + width, o_idx, o_val, nnz, ws,
                          dense_out=dense, capacity=cap)
    torch.cuda.synchronize()
    assert nnz.tolist() == [U, U]
    assert np.array_equal(o_idx.cpu().numpy().view(np.uint32)[:U], ref["idx"])
    want = ref["val"].astype(np.float32)
    assert np.array_equal(o_val.cpu().numpy()[:U], want)
    full = np.zeros(width, np.float32)
    full[ref["idx"].astype(np.int64) - lo] = want
    assert np.array_equal(dense.cpu().numpy(), full)


@pytest.mark.parametrize("P,share,least", [(2, 0.05, 0.09), (8, 0.1, 0.0835), (8, 0.7, 0.46), (33, 0.2, 0.125), (64, 0.05, 0.056)])
@pytest.mark.parametrize("B", [1, 40])
def test_less_workspace_than_told(B, P, share, least):
    """From the table of the tiles of a region hit evenly on, any workspace does: the
    same results, whatever tiles it has room for.  Below it the call is refused."""
    rng = np.random.default_rng(P)
    width = 700_001
    regions = [(b * 13, b * 13 + width, [some(rng, b * 13, width, 2_000 if b in (0, B - 1) else 3) for _ in range(P)])
               for b in range(B)]
    for ws_share in (1.0, 0.5, least):
        run_batch(regions, P, width, int(share * width), ws_share=ws_share)
    with pytest.raises(okt.OktError):
        run_batch(regions, P, width, int(share * width), ws_share=0.5 * least)
