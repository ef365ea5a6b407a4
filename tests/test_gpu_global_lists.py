"""The global stage's calls on short lists, at the lengths where their kernels change
form: the COO select in one workgroup, by tiles, and through the chained scan; the
intersection with a global list that is searched in one, two or more steps, with and
without room for the first launch's bits.  Everything is bit-exact.
"""
import numpy as np
import pytest
import torch

import paper_2201_07598_amd as okt
from oracle import okt_oracle as orc
from tests.okt_harness import DEV, bits_equal, to_dev, u32, u64, workspace

pytestmark = pytest.mark.gpu


def ascending(rng, space, count):
    return np.sort(rng.choice(space, count, replace=False)).astype(np.uint32)


def intersect(acc, local, glob, zero, ws_bytes, slack=3):
    residual = acc.copy()
    if not zero:
        residual[local] = 0.0
    d_res = to_dev(residual)
    d_local = to_dev(np.concatenate([local, np.zeros(slack, np.uint32)]))
    d_val = to_dev(np.concatenate([acc[local], np.full(slack, 9.0, np.float32)]))
    d_glob = to_dev(np.concatenate([glob, np.full(1, 7, np.uint32)]))
    d_nl, d_ng = (to_dev(np.array([a.size], np.uint64)) for a in (local, glob))
    out = torch.full((local.size + slack,), -1, dtype=torch.int32, device=DEV)
    cnt = torch.full((1,), -5, dtype=torch.int64, device=DEV)
    ws = workspace(ws_bytes)[:ws_bytes]
    kw = dict(indexes_out=out, max_local=local.size + slack, max_global=glob.size)
    if zero:
        okt.okt_index_intersect_zero(d_res, d_local, d_nl, d_glob, d_ng, cnt, ws, **kw)
    else:
        okt.okt_index_intersect_restore(d_res, d_local, d_val, d_nl, d_glob, d_ng, cnt, ws, **kw)
    c = int(u64(cnt)[0])
    return d_res.cpu().numpy(), u32(out[:c])


def least_bytes(max_local):
    tiles = max(1, -(-max_local // 1024))
    return 64 + 8 * (tiles + (tiles + 63) // 64)


# 1024 places of the global list are searched first; up to 16 elements between two of
# them are read at once (17 x 1024 = 17,408), of longer lists the part that a tile lies
# in, which fits in LDS up to 4096, else is sampled, and bisected from 17 x 4096 on
@pytest.mark.parametrize("ng", [1, 1023, 1024, 1025, 2048, 17_407, 17_408, 17_409, 60_000, 400_000])
@pytest.mark.parametrize("small_ws", [False, True])
@pytest.mark.parametrize("zero", [False, True])
def test_intersection_at_the_steps_of_the_search(ng, small_ws, zero):
    rng = np.random.default_rng(ng)
    n = 1_200_000
    acc = rng.normal(size=n).astype(np.float32)
    glob = ascending(rng, n, ng)
    # a crowded stretch, a sparse one whose tile spans most of the global list, the very ends
    crowd = np.arange(n // 2, n // 2 + 3000, dtype=np.uint32)
    local = np.unique(np.concatenate([crowd, glob[::5], ascending(rng, n, 700),
                                      np.array([0, n - 1], np.uint32)])).astype(np.uint32)
    nbytes = least_bytes(local.size + 3) if small_ws else okt.okt_workspace_bytes(local.size + 3, 0)
    got, indexes = intersect(acc, local, glob, zero, nbytes)
    want = orc.index_intersection(local, glob)
    assert np.array_equal(indexes, want)
    assert bits_equal(got, orc.residual_update(acc, want))


def test_intersection_of_a_sparse_tile_with_a_long_list():
    """One tile of local entries over a list of 3 M: sampled in LDS, then bisected."""
    rng = np.random.default_rng(5)
    n = 9_000_000
    acc = rng.normal(size=n).astype(np.float32)
    glob = ascending(rng, n, 3_000_000)
    local = np.unique(np.concatenate([rng.choice(glob, 500), ascending(rng, n, 400)])).astype(np.uint32)
    got, indexes = intersect(acc, local, glob, True, okt.okt_workspace_bytes(local.size + 3, 0))
    want = orc.index_intersection(local, glob)
    assert np.array_equal(indexes, want)
    assert bits_equal(got, orc.residual_update(acc, want))


# a few tiles, and more than run at a time
@pytest.mark.parametrize("nl,ng", [(900, 1_300), (5_000, 7_000), (700_000, 900_000)])
@pytest.mark.parametrize("over", ["local", "global", "counts"])
@pytest.mark.parametrize("zero", [False, True])
def test_intersection_written_over_its_input(nl, ng, over, zero):
    """The matched indices take the place of the local or the global list, the count that of
    an input's count."""
    rng = np.random.default_rng(nl)
    n = 2_000_000
    acc = rng.normal(size=n).astype(np.float32)
    local, glob = ascending(rng, n, nl), ascending(rng, n, ng)
    want = orc.index_intersection(local, glob)
    residual = acc.copy()
    if not zero:
        residual[local] = 0.0
    d_res, d_val = to_dev(residual), to_dev(acc[local])
    d_local, d_glob = to_dev(local), to_dev(glob)
    d_nl, d_ng = (to_dev(np.array([a.size], np.uint64)) for a in (local, glob))
    out = {"local": d_local, "global": d_glob}.get(over)
    if out is None:
        out = torch.full((nl,), -1, dtype=torch.int32, device=DEV)
    cnt = d_nl if over != "global" else d_ng
    ws = workspace(okt.okt_workspace_bytes(nl, 0))
    if zero:
        okt.okt_index_intersect_zero(d_res, d_local, d_nl, d_glob, d_ng, cnt, ws, indexes_out=out)
    else:
        okt.okt_index_intersect_restore(d_res, d_local, d_val, d_nl, d_glob, d_ng, cnt, ws, indexes_out=out)
    assert int(u64(cnt)[0]) == want.size
    assert np.array_equal(u32(out[:want.size]), want)
    assert bits_equal(d_res.cpu().numpy(), orc.residual_update(acc, want))


def test_intersection_waits_that_give_up_are_reported():
    """The least workspace has no room for a bit per entry: places come from a scan across
    workgroups, whose waits are limited to one poll here.  A call completes or reports
    UINT64_MAX; it never hangs.  More tiles than workgroups are launched."""
    rng = np.random.default_rng(7)
    n = 2_000_000
    acc = rng.normal(size=n).astype(np.float32)
    local, glob = ascending(rng, n, 700_000), ascending(rng, n, 900_000)
    want = orc.index_intersection(local, glob)
    d_res, d_local, d_glob = to_dev(acc), to_dev(local), to_dev(glob)
    d_nl, d_ng = (to_dev(np.array([a.size], np.uint64)) for a in (local, glob))
    out = torch.full((local.size,), -1, dtype=torch.int32, device=DEV)
    ws = workspace(least_bytes(local.size))[:least_bytes(local.size)]
    for limit in (1, 0):
        okt.okt_debug_spin_limit(limit)
        try:
            for _ in range(3):
                cnt = torch.full((1,), -5, dtype=torch.int64, device=DEV)
                okt.okt_index_intersect_zero(d_res, d_local, d_nl, d_glob, d_ng, cnt, ws, indexes_out=out)
                torch.cuda.synchronize()
                c = int(u64(cnt)[0])
                if limit == 0 or c != 0xFFFFFFFFFFFFFFFF:
                    assert c == want.size and np.array_equal(u32(out[:c]), want)
        finally:
            okt.okt_debug_spin_limit(0)
    assert bits_equal(d_res.cpu().numpy(), orc.residual_update(acc, want))


def test_intersection_of_more_tiles_than_are_added_up():
    """More than 4096 tiles of room: the counts are made prefixes by a launch of their own."""
    rng = np.random.default_rng(6)
    n = 6_000_000
    acc = rng.normal(size=n).astype(np.float32)
    local = ascending(rng, n, 4_300_000)
    glob = ascending(rng, n, 900_000)
    got, indexes = intersect(acc, local, glob, False, okt.okt_workspace_bytes(local.size + 3, 0))
    want = orc.index_intersection(local, glob)
    assert np.array_equal(indexes, want)
    assert bits_equal(got, orc.residual_update(acc, want))


@pytest.mark.parametrize("nnz", [4, 1023, 16_384, 16_385, 32_768, 32_769, 33_793, 4 << 20, (4 << 20) + 1])
@pytest.mark.parametrize("slack", [0, 5])
def test_coo_select_at_the_lengths_of_its_forms(nnz, slack):
    rng = np.random.default_rng(nnz)
    idx = np.cumsum(rng.integers(1, 9, nnz), dtype=np.uint64).astype(np.uint32)
    val = rng.normal(size=nnz).astype(np.float32)
    val[::211] = np.float32(np.nan)
    th = np.float32(1.1)
    # the indices at an odd word address, garbage behind the entries there are
    store = to_dev(np.concatenate([np.zeros(1, np.uint32), idx, np.full(slack, 3, np.uint32)]))[1:]
    d_val = to_dev(np.concatenate([val, np.full(slack, 1e30, np.float32)]))
    ws_bytes = 64 + 8 * (nnz // 262_144 + 1025 + (nnz // 262_144 + 1025 + 63) // 64) + 16
    want_idx, want_val, total = orc.coo_threshold_select(idx, val, th)
    for cap in (nnz + slack, total // 2):
        out_idx = torch.full((nnz + slack,), -1, dtype=torch.int32, device=DEV)
        out_val = torch.zeros(nnz + slack, device=DEV)
        out_nnz = torch.zeros(2, dtype=torch.int64, device=DEV)
        okt.okt_coo_threshold_select(store, d_val, to_dev(np.array([nnz], np.uint64)), to_dev(np.array([th])),
                                     out_idx, out_val, out_nnz, workspace(ws_bytes)[:ws_bytes],
                                     max_nnz=nnz + slack, capacity=cap)
        emitted, found = (int(x) for x in u64(out_nnz))
        assert found == total and emitted == min(cap, total)
        assert np.array_equal(u32(out_idx[:emitted]), want_idx[:emitted])
        assert bits_equal(out_val[:emitted].cpu().numpy(), want_val[:emitted])
        assert bool((out_idx[emitted:] == -1).all())


@pytest.mark.parametrize("nnz,over", [(3_000, "all"), (32_768, "all"), (40_000, "counts"), (40_000, "values"),
                                      (600_000, "counts"), (600_000, "values")])
def test_coo_select_written_over_its_input(nnz, over):
    """The counts, the values or, in a list that one workgroup selects, all outputs take the
    place of their inputs."""
    rng = np.random.default_rng(nnz)
    idx = np.cumsum(rng.integers(1, 9, nnz), dtype=np.uint64).astype(np.uint32)
    val = rng.normal(size=nnz).astype(np.float32)
    th = np.float32(1.1)
    want_idx, want_val, total = orc.coo_threshold_select(idx, val, th)
    d_th, ws = to_dev(np.array([th])), workspace(okt.okt_workspace_bytes(nnz, 0))
    for _ in range(5):
        d_idx, d_val, d_nnz = to_dev(idx), to_dev(val), to_dev(np.array([nnz, nnz], np.uint64))
        out_idx = d_idx if over == "all" else torch.full((nnz,), -1, dtype=torch.int32, device=DEV)
        out_val = d_val if over != "counts" else torch.zeros(nnz, device=DEV)
        out_nnz = d_nnz if over != "values" else torch.zeros(2, dtype=torch.int64, device=DEV)
        okt.okt_coo_threshold_select(d_idx, d_val, d_nnz, d_th, out_idx, out_val, out_nnz, ws)
        assert [int(x) for x in u64(out_nnz)] == [total, total]
        assert np.array_equal(u32(out_idx[:total]), want_idx) and bits_equal(out_val[:total].cpu().numpy(), want_val)
