"""GPU parity at the full sizes of the five configurations, through the same
entry points and launch shapes bench.py times.  The oracle checks every element
of every iteration (numpy handles these lengths in seconds): cfg2's ten
iterations, cfg4's three, and cfg3 through its second threshold re-evaluation
(iterations 0 to 32: the refresh at iteration 32 runs on a residual carried for
31 iterations of a reused threshold)."""
import numpy as np
import pytest
import torch

import paper_2201_07598_amd as okt
import workloads as wl
from oracle import okt_oracle as orc
from tests import sample_replay as sr
from tests.okt_harness import (DEV, GpuPath, bits_equal, gpu_reduce, reduce_tolerance, to_dev,
                               u32, u64, workspace)

pytestmark = pytest.mark.gpu


def loop(w, iterations, fused=False, capsys=None):
    """fused: as bench.py's step does, the iterations that re-evaluate the
    threshold take okt_accumulate_topk_select and those that reuse it
    okt_accumulate_select.  With capsys the per-iteration line goes to the real
    stdout (a long schedule must not look hung to whoever watches the run)."""
    import contextlib
    gpu = GpuPath(w.n, 4 * w.k)
    res = np.zeros(w.n, dtype=np.float32)
    th = None
    ridx = None
    for it in range(iterations):
        g = wl.gradient(w, it)
        acc = orc.residual_accumulate(g, res, w.lr)
        if fused and w.refresh(it):
            okt.okt_accumulate_topk_select(to_dev(g), gpu.residual, w.lr, w.k, gpu.th, gpu.count_ge,
                                           gpu.idx, gpu.val, gpu.nnz, gpu.ws, capacity=gpu.capacity)
            del g
            th, cnt = orc.topk_threshold_exact(acc, w.k, method="partition")
            assert gpu.th.cpu().numpy().view(np.uint32)[0] == np.float32(th).view(np.uint32), it
            assert int(u64(gpu.count_ge)[0]) == cnt, it
        elif fused:
            okt.okt_accumulate_select(to_dev(g), gpu.residual, w.lr, gpu.th, gpu.idx, gpu.val,
                                      gpu.nnz, gpu.ws, capacity=gpu.capacity)
            del g
        else:
            gpu.accumulate(to_dev(g), w.lr)
            del g
            if w.refresh(it):
                gpu.threshold(w.k)
                th, cnt = orc.topk_threshold_exact(acc, w.k, method="partition")
                assert gpu.th.cpu().numpy().view(np.uint32)[0] == np.float32(th).view(np.uint32), it
                assert int(u64(gpu.count_ge)[0]) == cnt, it
            gpu.select()
        ridx, rval, res, total = orc.threshold_select(acc, th, capacity=4 * w.k)
        del acc
        idx, val, emitted, gtotal = gpu.selected()
        assert (emitted, gtotal) == (ridx.size, total), it
        assert np.array_equal(idx, ridx) and bits_equal(val, rval), it
        assert bits_equal(gpu.residual.cpu().numpy(), res), it
        if w.refresh(it):
            assert total == cnt
        with capsys.disabled() if capsys is not None else contextlib.nullcontext():
            print(f"{w.name} it={it} nnz={total} |nnz-k|/k={abs(total - w.k) / w.k:.4f}", flush=True)
    return gpu, ridx


def check_partition(gpu, ridx, n, R):
    b = torch.zeros(R + 1, dtype=torch.int32, device=DEV)
    off = torch.zeros(R + 1, dtype=torch.int64, device=DEV)
    okt.okt_region_partition(gpu.idx, gpu.nnz, n, R, b, off)
    rb, roff = orc.region_partition(ridx, n, R)
    assert np.array_equal(u32(b), rb) and np.array_equal(u64(off), roff)
    return rb


def check_reduce(idx, val, off, lo, hi):
    got = gpu_reduce(idx, val, off, lo, hi)
    ref = orc.sparse_reduce(idx, val, off, lo, hi)
    assert got["total"] == got["emitted"] == ref["idx"].size
    assert np.array_equal(got["idx"], ref["idx"])
    err = np.abs(got["val"].astype(np.float64) - ref["val"].astype(np.float64))
    assert np.all(err <= reduce_tolerance(ref))
    tol = np.zeros(hi - lo)
    tol[ref["idx"].astype(np.int64) - lo] = reduce_tolerance(ref)
    assert np.all(np.abs(got["dense"].astype(np.float64) - ref["dense"]) <= tol)
    return ref


@pytest.mark.timeout(300)
def test_cfg2_full_size():
    w = wl.WORKLOADS["cfg2"]
    gpu, ridx = loop(w, 3)                      # exact threshold at 0, reused at 1 and 2
    check_partition(gpu, ridx, w.n, w.P)
    lo, hi = 0, w.n // w.P                      # the region bench.py reduces
    ref = check_reduce(*wl.contributions(w, lo, hi), lo, hi)
    assert ref["idx"].size > 0.9 * w.P * w.m


@pytest.mark.timeout(800)
@pytest.mark.parametrize("name,iterations", [("cfg2", 10), ("cfg3", 33), ("cfg4", 3)])
def test_full_size_full_schedule(name, iterations, capsys):
    """The schedule bench.py times, at full length: one call per iteration -
    okt_accumulate_topk_select where Alg.1 re-evaluates the threshold (0-based
    iteration it with it mod tau' = 0: cfg2 at 0, cfg3 at 0 and 32, cfg4 always),
    okt_accumulate_select where it reuses it - with threshold, count, index set,
    values and the whole residual compared with the oracle after every iteration.
    The layered vectors select whole layers (the stash-overflow path at full size)."""
    w = wl.WORKLOADS[name]
    assert [it for it in range(iterations) if w.refresh(it)] == \
        {"cfg2": [0], "cfg3": [0, 32], "cfg4": [0, 1, 2]}[name]
    loop(w, iterations, fused=True, capsys=capsys)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("name", ["cfg2", "cfg5"])
def test_reduce_batch_at_the_size_the_bench_times(name):
    """The batched reduce as bench.py launches it: B regions of the workload's
    shape in one call, more than 1 GB of input (490 regions at cfg2).  Every
    region's count is checked against the union size of its index pattern, and
    sampled regions - the first, the last, some in between - entry by entry
    against the oracle."""
    w = wl.WORKLOADS[name]
    P, m, width = w.P, w.m, w.n // w.P
    E1 = P * m
    B = int(1.0e9 // (8 * E1)) + 1
    base_sets = min(B, 32)
    sets = [wl.contributions(w, 0, width, stream=1000 + s) for s in range(base_sets)]
    assert all(ci.size == E1 for ci, _, _ in sets)
    idx_cat = np.empty(B * E1, dtype=np.uint32)
    off = np.empty(B * (P + 1), dtype=np.uint64)
    lohi = np.empty(2 * B, dtype=np.uint32)
    for j in range(B):
        ci, _, co = sets[j % base_sets]
        rlo = j * width
        if rlo + width > 0xFFFFFFFF:
            rlo = (j % 16) * width
        idx_cat[j * E1:(j + 1) * E1] = ci + np.uint32(rlo)
        off[j * (P + 1):(j + 1) * (P + 1)] = co + np.uint64(j * E1)
        lohi[2 * j], lohi[2 * j + 1] = rlo, rlo + width
    val_cat = np.random.default_rng(4242).standard_normal(B * E1, dtype=np.float32) * np.float32(1e-3)
    out_idx = torch.full((B * E1,), -1, dtype=torch.int32, device=DEV)
    out_val = torch.zeros(B * E1, dtype=torch.float32, device=DEV)
    nnz = torch.zeros(2 * B, dtype=torch.int64, device=DEV)
    ws = workspace(okt.okt_sparse_reduce_batch_workspace_bytes(B, P, width))
    okt.okt_sparse_reduce_batch(to_dev(idx_cat), to_dev(val_cat), to_dev(off), to_dev(lohi), B, P,
                                width, out_idx, out_val, E1, nnz, ws)
    torch.cuda.synchronize()
    counts = u64(nnz).reshape(B, 2)
    unions = [np.unique(ci).size for ci, _, _ in sets]
    assert np.array_equal(counts[:, 0], counts[:, 1])
    assert np.array_equal(counts[:, 1], np.array([unions[j % base_sets] for j in range(B)], dtype=np.uint64))
    print(f"{name}: B={B} regions, {B * E1} entries in, {int(counts[:, 1].sum())} out", flush=True)
    for j in sorted({0, 1, base_sets - 1, base_sets, B // 2, B - 2, B - 1}):
        lo, hi = int(lohi[2 * j]), int(lohi[2 * j + 1])
        sl = slice(j * E1, (j + 1) * E1)
        ref = orc.sparse_reduce(idx_cat[sl], val_cat[sl], off[j * (P + 1):(j + 1) * (P + 1)] - np.uint64(j * E1), lo, hi)
        U = ref["idx"].size
        assert U == int(counts[j, 1]), j
        assert np.array_equal(u32(out_idx[j * E1:j * E1 + U]), ref["idx"]), j
        err = np.abs(out_val[j * E1:j * E1 + U].cpu().numpy().astype(np.float64) - ref["val"])
        assert np.all(err <= reduce_tolerance(ref)), j


@pytest.mark.timeout(300)
def test_cfg3_full_size():
    w = wl.WORKLOADS["cfg3"]
    gpu, ridx = loop(w, 2)
    rb = check_partition(gpu, ridx, w.n, w.P)
    lo, hi = w.n // w.P, 2 * (w.n // w.P)
    ref = check_reduce(*wl.contributions(w, lo, hi), lo, hi)
    # 30 % of each worker's entries are one shared pool: they collide P ways
    assert ref["hits"].max() == w.P and int(ref["idx"].size) < w.P * w.m


@pytest.mark.timeout(600)
def test_cfg4_full_size():
    w = wl.WORKLOADS["cfg4"]
    gpu, ridx = loop(w, 2)                      # exact radix select in both iterations
    rb = check_partition(gpu, ridx, w.n, 64).astype(np.int64)
    widths = np.diff(rb)
    r = int(np.argmax(widths))                  # the widest region
    lo, hi = int(rb[r]), int(rb[r + 1])
    check_reduce(*wl.contributions(w, lo, hi), lo, hi)


@pytest.mark.timeout(300)
def test_cfg5_full_size():
    w = wl.WORKLOADS["cfg5"]
    width = -(-w.n // w.P)                      # one GPU's region of a 256-GPU job
    lo = 128 * width
    idx, val, off = wl.contributions(w, lo, lo + width)
    ref = check_reduce(idx, val, off, lo, lo + width)
    assert ref["hits"].max() > 64               # hot indices collide across most workers


@pytest.mark.timeout(600)
def test_longest_vector_the_interface_allows():
    """n = 2^32 - 1, the largest length the 32-bit indices address: a vector of
    zeros with a few thousand planted entries - at both ends, around the
    boundaries of pieces and tiles, and at random - so that every index the
    kernels form near 2^32 matters.  Zeros can never be selected (the threshold
    is positive), so the oracle runs on the planted entries alone, whose order is
    the order of their positions."""
    n = (1 << 32) - 1
    rng = np.random.default_rng(77)
    special = [0, 1, 2, 3, 4, 255, 256, 257, 1023, 1024, 16383, 16384, 16385,
               n - 1, n - 2, n - 3, n - 4, n - 5, n - 255, n - 256, n - 257, n - 1024, n - 1025,
               (1 << 31) - 1, 1 << 31, (1 << 31) + 1]
    special += [j * 16384 * 16 + d for j in (1, 7, 4095, 16383) for d in (-1, 0, 1)]
    pos = np.unique(np.concatenate([np.array(special, dtype=np.int64),
                                    rng.integers(0, n, 3000, dtype=np.int64)]))
    pos = pos[(pos >= 0) & (pos < n)]
    m = pos.size

    def planted(seed):
        r = np.random.default_rng(seed)
        mag = 1.0 + r.permutation(m).astype(np.float64) / 4096.0       # distinct magnitudes
        return (mag * r.choice([-1.0, 1.0], m)).astype(np.float32)

    d_pos = torch.from_numpy(pos).to(DEV)
    gpu = GpuPath(n, 4096)
    grad = torch.zeros(n, dtype=torch.float32, device=DEV)
    lr, k = 0.5, 500
    g_c, e_c = planted(1), (planted(2) * np.float32(0.25)).astype(np.float32)
    grad[d_pos] = torch.from_numpy(g_c).to(DEV)
    gpu.residual[d_pos] = torch.from_numpy(e_c).to(DEV)

    # iteration 0: accumulate, exact threshold, select, partition
    gpu.accumulate(grad, lr)
    acc_c = orc.residual_accumulate(g_c, e_c, lr)
    assert np.count_nonzero(acc_c) == m
    assert bits_equal(gpu.residual[d_pos].cpu().numpy(), acc_c)
    assert int(torch.count_nonzero(gpu.residual)) == m
    print("accumulate ok", flush=True)
    gpu.threshold(k)
    th, cnt = orc.topk_threshold_exact(acc_c, k)
    assert gpu.th.cpu().numpy().view(np.uint32)[0] == np.float32(th).view(np.uint32)
    assert int(u64(gpu.count_ge)[0]) == cnt == k
    print("threshold ok", flush=True)
    gpu.select()
    ridx_c, rval, res_c, total = orc.threshold_select(acc_c, th, capacity=gpu.capacity)
    idx, val, emitted, gtotal = gpu.selected()
    assert (emitted, gtotal) == (ridx_c.size, total) == (k, k)
    assert np.array_equal(idx.astype(np.int64), pos[ridx_c]) and bits_equal(val, rval)
    assert bits_equal(gpu.residual[d_pos].cpu().numpy(), res_c)
    assert int(torch.count_nonzero(gpu.residual)) == np.count_nonzero(res_c)
    print("select ok", flush=True)
    check_partition(gpu, pos[ridx_c].astype(np.uint32), n, 64)

    # iteration 1: the same threshold, accumulate and select in one pass; then a
    # threshold below everything planted, which overflows the output
    g2_c = planted(3)
    grad[d_pos] = torch.from_numpy(g2_c).to(DEV)
    okt.okt_accumulate_select(grad, gpu.residual, lr, gpu.th, gpu.idx, gpu.val, gpu.nnz, gpu.ws,
                              capacity=gpu.capacity)
    acc_c = orc.residual_accumulate(g2_c, res_c, lr)
    ridx_c, rval, res_c, total = orc.threshold_select(acc_c, th, capacity=gpu.capacity)
    idx, val, emitted, gtotal = gpu.selected()
    assert (emitted, gtotal) == (ridx_c.size, total)
    assert np.array_equal(idx.astype(np.int64), pos[ridx_c]) and bits_equal(val, rval)
    assert bits_equal(gpu.residual[d_pos].cpu().numpy(), res_c)
    assert int(torch.count_nonzero(gpu.residual)) == np.count_nonzero(res_c)
    print("accumulate+select ok", flush=True)
    low = np.float32(1e-3)
    gpu.th.fill_(float(low))
    okt.okt_threshold_select_copy(gpu.residual, gpu.th, gpu.idx, gpu.val, gpu.nnz, gpu.ws,
                                  capacity=1000)
    ridx_c, rval, _, total = orc.threshold_select(res_c, low, capacity=1000)
    idx, val, emitted, gtotal = gpu.selected()
    assert (emitted, gtotal) == (1000, total) and total > 1000
    assert np.array_equal(idx.astype(np.int64), pos[ridx_c]) and bits_equal(val, rval)
    assert bits_equal(gpu.residual[d_pos].cpu().numpy(), res_c)          # left untouched
    print("select without zeroing ok", flush=True)

    # a refresh iteration in one call from a fresh residual.  Small entries are planted where
    # the threshold's sample looks, twenty for each of its workgroups, so that every bound is
    # a positive value below the others and the call's one-pass path - candidates collected,
    # selection over them - runs at this n
    del grad
    runs = np.concatenate([wg + sr.WORKGROUPS * rng.choice(sr.RUNS // sr.WORKGROUPS, 20, replace=False)
                           for wg in range(sr.WORKGROUPS)])
    pos_s = sr.run_starts(n)[runs].astype(np.int64) + rng.integers(0, sr.RUN, runs.size)
    pos_s = np.setdiff1d(pos_s, pos)
    pos2 = np.concatenate([pos, pos_s])
    order = np.argsort(pos2, kind="stable")
    g3_c = np.concatenate([planted(4), (0.25 + rng.random(pos_s.size) / 16).astype(np.float32)])
    pos2, g3_c = pos2[order], g3_c[order]
    d_pos2 = torch.from_numpy(pos2).to(DEV)
    gpu.residual.zero_()
    grad = torch.zeros(n, dtype=torch.float32, device=DEV)
    grad[d_pos2] = torch.from_numpy(g3_c).to(DEV)
    keys = sr.key_of(orc.residual_accumulate(g3_c, np.zeros_like(g3_c), lr))
    bounds = sr.bounds(n, k, pos2, keys)
    passing = int(np.count_nonzero(keys >= bounds.min()))
    assert bounds.min() > 0 and k <= passing
    okt.okt_accumulate_topk_select(grad, gpu.residual, lr, k, gpu.th, gpu.count_ge, gpu.idx, gpu.val,
                                   gpu.nnz, gpu.ws, capacity=gpu.capacity)
    state = sr.State(gpu.ws)
    assert np.array_equal(state.bounds, bounds) and state.collected == passing
    acc_c = orc.residual_accumulate(g3_c, np.zeros_like(g3_c), lr)
    th, cnt = orc.topk_threshold_exact(acc_c, k)
    assert gpu.th.cpu().numpy().view(np.uint32)[0] == np.float32(th).view(np.uint32)
    assert int(u64(gpu.count_ge)[0]) == cnt == k
    ridx_c, rval, res_c, total = orc.threshold_select(acc_c, th, capacity=gpu.capacity)
    idx, val, emitted, gtotal = gpu.selected()
    assert (emitted, gtotal) == (ridx_c.size, total) == (k, k)
    assert np.array_equal(idx.astype(np.int64), pos2[ridx_c]) and bits_equal(val, rval)
    assert bits_equal(gpu.residual[d_pos2].cpu().numpy(), res_c)
    assert int(torch.count_nonzero(gpu.residual)) == np.count_nonzero(res_c)
    print("refresh iteration in one call ok", flush=True)
