"""What the speed of this library is measured on.

A case is one pass of a worker's work on one GPU, through the calls of the Python
binding, with everything resident in device memory before the pass:

  step      a whole iteration that re-evaluates the threshold: accumulate, exact
            threshold and select in one call, the balanced partition, the reduce of
            the own region, the global threshold over the reduced values, the
            global select, and the residual put right afterwards
  refresh   okt_accumulate_topk_select alone: the dense part of such an iteration
  reuse     okt_accumulate_select: the dense part of the iterations in between
  separate  the same made of its three calls (okt_residual_accumulate,
            okt_topk_threshold_exact, okt_threshold_select)
  literal   an iteration that zeroes the residual after the allreduce only:
            accumulate, select without zeroing, global threshold, global select,
            intersection and zeroing
  region    okt_sparse_reduce: one region, with its dense copy
  batch     okt_sparse_reduce_batch: many regions in one launch

The gradients of a state are a ring of RING vectors that sum to zero, taken in turn:
noise around zero, as a stochastic gradient is, but finite.  A residual that meets
fresh noise settles into a steady state; under this ring it settles into one that
repeats, so that every pass over a state selects as much as the one before, however
many there are (0.7 to 1.0 k with a threshold that is reused, k with an exact one).
The residual a state starts from has been through BURN_IN iterations.
"""
import math
import random

import numpy as np
import torch

import paper_2201_07598_amd as okt

DEV = "cuda:0"
RING = 3
BURN_IN = 9                     # a whole number of turns of the ring
LR = 0.1
PIECE = 1 << 26                 # elements drawn at a time


def listed():
    return [
        # the smallest iteration: 1 Mi iid elements at 1 %, four workers; a dozen calls
        # whose launches and latencies are what counts
        {"name": "step_1m", "kind": "step", "n": 1_048_576, "per_mille": 10, "dist": "laplace",
         "layers": 0, "P": 4},
        # the same length on an iteration that reuses its threshold
        {"name": "reuse_1m", "kind": "reuse", "n": 1_048_576, "per_mille": 10, "dist": "laplace",
         "layers": 0},
        # VGG-16: its 14,728,266 parameters at the 2 % it is trained with
        {"name": "refresh_14m", "kind": "refresh", "n": 14_728_266, "per_mille": 20,
         "dist": "normal", "layers": 161},
        # LSTM: 27,569,568 parameters at 2 %, the iterations between two thresholds
        {"name": "reuse_27m", "kind": "reuse", "n": 27_569_568, "per_mille": 20, "dist": "normal",
         "layers": 161},
        # a ResNet-50-sized layered gradient, the iteration spelled as the paper does
        {"name": "literal_25m", "kind": "literal", "n": 25_557_032, "per_mille": 10,
         "dist": "normal", "layers": 161, "P": 16},
        # BERT-base-sized, layered, 1 %: most iterations of the training
        {"name": "reuse_110m", "kind": "reuse", "n": 110_000_000, "per_mille": 10,
         "dist": "laplace", "layers": 199},
        # BERT: 133,547,324 parameters, an iteration made of the separate calls
        {"name": "separate_133m", "kind": "separate", "n": 133_547_324, "per_mille": 10,
         "dist": "laplace", "layers": 199},
        # BERT-large-sized, heavy tails, 0.1 %, exact threshold every iteration
        {"name": "refresh_336m", "kind": "refresh", "n": 336_000_000, "per_mille": 1,
         "dist": "student3", "layers": 0},
        # one worker's region of 32: 3.4 M indices, 34,375 entries from each worker, 30 %
        # of them common to all
        {"name": "region_p32", "kind": "region", "P": 32, "width": 3_437_500, "m": 34_375,
         "contrib": "overlap30"},
        # regions in bulk: few long contributions, many short ones, and very many that
        # collide on the same hot indices
        {"name": "batch_p16", "kind": "batch", "B": 490, "P": 16, "width": 1_597_315, "m": 15_973,
         "contrib": "uniform"},
        {"name": "batch_p64", "kind": "batch", "B": 373, "P": 64, "width": 5_250_000, "m": 5_250,
         "contrib": "uniform"},
        {"name": "batch_p256", "kind": "batch", "B": 48, "P": 256, "width": 429_688, "m": 4_296,
         "contrib": "zipf"},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    """Lengths from 100,000 to 336 M and densities from 0.1 to 2 % in every form of the
    dense part; regions of 2 to 256 workers, from sparsely to densely hit."""
    kind = rng.choice(["step", "refresh", "refresh", "reuse", "reuse", "separate", "literal",
                       "region", "batch", "batch"])
    if kind in ("region", "batch"):
        contrib = rng.choice(["uniform", "overlap30", "zipf"])
        P = _log_uniform(rng, 2, 256)
        width = _log_uniform(rng, 20_000, 5_000_000 if contrib != "zipf" else 500_000)
        # of the region's indices, the share that all contributions together come to
        share = math.exp(rng.uniform(math.log(0.03), math.log(2.0)))
        m = max(16, int(width * share / P))
        c = {"kind": kind, "P": P, "width": width, "m": m, "contrib": contrib}
        if kind == "batch":
            entries = _log_uniform(rng, 1_000_000, 60_000_000)
            c["B"] = max(2, min(2000, entries // (P * m), 400_000_000 // width))
        return c
    top = {"step": 8_000_000, "literal": 110_000_000}.get(kind, 336_000_000)
    n = _log_uniform(rng, 100_000, top)
    dist = rng.choice(["normal", "laplace", "student3"])
    c = {"kind": kind, "n": n, "per_mille": rng.choice([1, 10, 20]), "dist": dist,
         "layers": rng.choice([0, 161, 199])}
    if kind in ("step", "literal"):
        c["P"] = rng.choice([4, 8, 16, 32])
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + stream) & 0x7FFFFFFFFFFFFFFF)
    return g


def _noise(out, dist, g):
    for a in range(0, out.numel(), PIECE):
        part = out[a:a + PIECE]
        part.normal_(generator=g)
        if dist == "laplace":
            part.copy_(torch.empty_like(part).exponential_(generator=g).copysign_(part))
        elif dist == "student3":
            chi = torch.zeros_like(part)
            for _ in range(3):
                chi.add_(torch.empty_like(part).normal_(generator=g).square_())
            part.div_(chi.div_(3.0).sqrt_())
    return out


def _layer_scale(case, seed):
    """Per-element scale of the layers: lengths over two decades, scales over three."""
    n, layers = case["n"], case["layers"]
    if not layers:
        return 1e-3
    r = np.random.default_rng([int(seed), 7])
    w = np.exp(r.uniform(math.log(0.1), math.log(10.0), layers))
    scale = np.exp(r.uniform(math.log(1e-5), math.log(1e-2), layers))
    length = 64 + np.floor(w / w.sum() * (n - 64 * layers)).astype(np.int64)
    length[-1] += n - length.sum()
    return torch.repeat_interleave(torch.from_numpy(scale.astype(np.float32)).to(DEV),
                                   torch.from_numpy(length).to(DEV), output_size=n)


def _k(case):
    return -(-case["n"] * case["per_mille"] // 1000)


def _kth_largest(mag, k):
    """The k-th largest of the magnitudes, exactly, by plain torch."""
    n = mag.numel()
    stride = max(1, n // (1 << 21))
    sample = mag[::stride]
    want = min(sample.numel(), int(1.3 * k / stride) + 64)
    top = mag[mag >= sample.kthvalue(sample.numel() - want + 1).values]
    if top.numel() < k:
        top = mag
    return top.sort(descending=True).values[k - 1]


def _accumulate(residual, grad):
    """eps + lr * G in fp32, product and sum rounded separately."""
    return residual + grad * np.float32(LR).item()


def _dense_state(case, seed):
    n, k = case["n"], _k(case)
    g = _gen(seed, 1)
    ring = [_noise(torch.empty(n, device=DEV), case["dist"], g) for _ in range(RING)]
    scale = _layer_scale(case, seed)
    mean = sum(ring[1:], ring[0].clone()).div_(RING)
    for x in ring:
        x.sub_(mean).mul_(scale)
    del mean, scale
    residual, th = torch.zeros(n, device=DEV), None
    for it in range(BURN_IN):
        acc = _accumulate(residual, ring[it % RING])
        mag = acc.abs()
        th = _kth_largest(mag, k)
        residual = acc.masked_fill_(mag >= th, 0.0)
    cap = min(n, 4 * k)
    return {
        "case": case, "n": n, "k": k, "at": 0, "ring": ring, "residual": residual,
        "th": th.reshape(1).clone(), "count": torch.zeros(1, dtype=torch.int64, device=DEV),
        "idx": torch.zeros(cap, dtype=torch.int32, device=DEV),
        "val": torch.zeros(cap, device=DEV),
        "nnz": torch.zeros(2, dtype=torch.int64, device=DEV),
        "ws": torch.empty(okt.okt_workspace_bytes(n, case.get("P", 1)), dtype=torch.uint8,
                          device=DEV),
    }


def _pack(rows):
    """Rows of ascending indices, negative where there is none -> (idx, counts)."""
    keep = rows >= 0
    return rows[keep].to(torch.int32), keep.sum(1)


def _spread(rows, m, width, g):
    """About m distinct ascending indices below `width` in each row, evenly spread."""
    gap = torch.empty(rows, m, device=DEV).exponential_(generator=g)
    at = gap.mul_(max(width / m - 0.5, 0.0)).to(torch.int32).add_(1).cumsum(1, dtype=torch.int64)
    return at.sub_(1).masked_fill_(at >= width, -1)


def _entries(contrib, regions, P, width, m, seed):
    """`regions` x P contributions: (idx, values, offsets uint64[regions * P + 1])."""
    g = _gen(seed, 2)
    parts, counts = [], []
    at_once = max(1, (1 << 25) // (P * m))
    if contrib == "zipf":
        pmf = np.arange(1, width + 1, dtype=np.float64) ** -1.1
        cdf = torch.from_numpy(np.cumsum(pmf) / pmf.sum()).to(DEV)
        perm = torch.randperm(width, device=DEV, generator=g)
    for a in range(0, regions, at_once):
        rows = min(at_once, regions - a) * P
        if contrib == "uniform":
            r = _spread(rows, m, width, g)
        elif contrib == "overlap30":
            # shared indices on the even places, private ones on the odd: no clash
            common, half = max(1, int(0.3 * m)), max(2, width // 2)
            pool = _spread(rows // P, common, half, g).repeat_interleave(P, 0)
            own = _spread(rows, max(1, m - common), half, g)
            r = torch.cat([torch.where(pool < 0, pool, 2 * pool),
                           torch.where(own < 0, own, 2 * own + 1)], 1).sort(1).values
        else:
            u = torch.rand(rows, 2 * m, device=DEV, generator=g, dtype=torch.float64)
            r = perm[torch.searchsorted(cdf, u, right=True).clamp_(max=width - 1)]
            r = r.sort(1).values
            r[:, 1:].masked_fill_(r[:, 1:] == r[:, :-1], -1)
        idx, cnt = _pack(r)
        parts.append(idx)
        counts.append(cnt)
    idx, cnt = torch.cat(parts), torch.cat(counts)
    off = torch.zeros(regions * P + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(cnt, 0, out=off[1:])
    val = torch.empty(idx.numel(), device=DEV).normal_(generator=g).mul_(1e-3)
    return idx, val, off


def _union(case):
    """The expected number of indices that at least one contribution of a region holds."""
    P, width, m = case["P"], case["width"], case["m"]
    if case["contrib"] == "uniform":
        return width * (1.0 - (1.0 - min(1.0, m / width)) ** P)
    if case["contrib"] == "overlap30":
        own = min(1.0, 1.4 * m / width)
        return 0.3 * m + width / 2 * (1.0 - (1.0 - own) ** P)
    pmf = np.arange(1, width + 1, dtype=np.float64) ** -1.1
    return float((1.0 - (1.0 - pmf / pmf.sum()) ** (2 * m * P)).sum())


def _entries_expected(case):
    if case["contrib"] != "zipf":
        return case["P"] * case["m"]
    pmf = np.arange(1, case["width"] + 1, dtype=np.float64) ** -1.1
    return case["P"] * float((1.0 - (1.0 - pmf / pmf.sum()) ** (2 * case["m"])).sum())


def _region_capacity(case):
    """Room for the case that nothing collides."""
    return int(1.02 * _entries_expected(case)) + 1024


def _region_state(case, seed):
    P, width = case["P"], case["width"]
    lo = 1_000 + width                                  # somewhere inside the index space
    idx, val, off = _entries(case["contrib"], 1, P, width, case["m"], seed)
    cap = _region_capacity(case)
    return {
        "case": case, "lo": lo, "hi": lo + width, "in_idx": idx.add_(lo), "in_val": val, "off": off,
        "idx": torch.zeros(cap, dtype=torch.int32, device=DEV), "val": torch.zeros(cap, device=DEV),
        "nnz": torch.zeros(2, dtype=torch.int64, device=DEV),
        "dense": torch.zeros(width, device=DEV),
        "ws": torch.empty(okt.okt_workspace_bytes(width, P), dtype=torch.uint8, device=DEV),
    }


def _batch_capacity(case):
    return min(case["width"], int(1.05 * _union(case)) + 64)


def _batch_state(case, seed):
    P, width, B = case["P"], case["width"], case["B"]
    idx, val, off = _entries(case["contrib"], B, P, width, case["m"], seed)
    # one region after the other in the index space, as far as 32 bits go
    apart = min(width, (2 ** 31 - 1 - width) // B)
    base = torch.arange(B, dtype=torch.int64, device=DEV) * apart
    length = (off[P::P] - off[:-1:P])
    idx += torch.repeat_interleave(base, length, output_size=idx.numel()).to(torch.int32)
    chunk = torch.cat([off[b * P:b * P + P + 1] for b in range(B)])
    lo_hi = torch.stack([base, base + width], 1).to(torch.int32).reshape(-1).contiguous()
    cap = _batch_capacity(case)
    return {
        "case": case, "in_idx": idx, "in_val": val, "off": chunk, "lo_hi": lo_hi, "cap": cap,
        "idx": torch.zeros(B * cap, dtype=torch.int32, device=DEV),
        "val": torch.zeros(B * cap, device=DEV),
        "nnz": torch.zeros(2 * B, dtype=torch.int64, device=DEV),
        "ws": torch.empty(okt.okt_sparse_reduce_batch_workspace_bytes(B, P, width),
                          dtype=torch.uint8, device=DEV),
    }


def _stage_after_reduce(s, case, seed, reduced):
    """Buffers of the global stage: the reduced region and the list that the allgatherv
    returns - some of what this worker selects, and as many again that it does not."""
    n, k, P = s["n"], s["k"], case["P"]
    g = _gen(seed, 3)
    acc = _accumulate(s["residual"], s["ring"][0])
    mine = (acc.abs() >= s["th"]).nonzero().reshape(-1)
    mine = mine[torch.rand(mine.numel(), device=DEV, generator=g) < 0.5]
    other = torch.randint(0, n, (k,), device=DEV, generator=g)
    glob = torch.unique(torch.cat([mine, other]))
    s.update({
        "k_global": max(1, reduced // 3), "max_reduced": reduced,
        "gth": torch.zeros(1, device=DEV), "gcount": torch.zeros(1, dtype=torch.int64, device=DEV),
        "gidx": torch.zeros(reduced, dtype=torch.int32, device=DEV),
        "gval": torch.zeros(reduced, device=DEV),
        "gnnz": torch.zeros(2, dtype=torch.int64, device=DEV),
        "all_idx": glob.to(torch.int32),
        "all_nnz": torch.tensor([glob.numel()], dtype=torch.int64, device=DEV),
        "common": torch.zeros(s["idx"].numel(), dtype=torch.int32, device=DEV),
        "ncommon": torch.zeros(1, dtype=torch.int64, device=DEV),
    })


def _own_region(case):
    """What the other workers send for one region of n / P indices."""
    width = case["n"] // case["P"]
    return {"kind": "region", "P": case["P"], "width": width,
            "m": max(16, _k(case) // case["P"]), "contrib": "uniform"}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "region":
        return _region_state(case, seed)
    if kind == "batch":
        return _batch_state(case, seed)
    s = _dense_state(case, seed)
    if kind == "step":
        r = _region_state(_own_region(case), seed)
        s.update({"reduce": r, "R": case["P"],
                  "bounds": torch.zeros(case["P"] + 1, dtype=torch.int32, device=DEV),
                  "offsets": torch.zeros(case["P"] + 1, dtype=torch.int64, device=DEV)})
        _stage_after_reduce(s, case, seed, r["idx"].numel())
    elif kind == "literal":
        # the reduced values of the own region, as the reduce left them
        size = max(16, _k(case))
        idx, val, _ = _entries("uniform", 1, 1, case["n"] // case["P"], size, seed)
        pad = (0, size - idx.numel())                  # the buffers have room for all of them
        s.update({"red_idx": torch.nn.functional.pad(idx, pad),
                  "red_val": torch.nn.functional.pad(val, pad),
                  "red_nnz": torch.tensor([idx.numel()], dtype=torch.int64, device=DEV)})
        _stage_after_reduce(s, case, seed, size)
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _next_grad(s):
    g = s["ring"][s["at"]]
    s["at"] = (s["at"] + 1) % RING
    return g


def run(s):
    kind = s["case"]["kind"]
    if kind == "region":
        okt.okt_sparse_reduce(s["in_idx"], s["in_val"], s["off"], s["lo"], s["hi"], s["idx"],
                              s["val"], s["nnz"], s["ws"], dense_out=s["dense"])
        return {"idx": s["idx"], "val": s["val"], "nnz": s["nnz"], "dense": s["dense"]}
    if kind == "batch":
        c = s["case"]
        okt.okt_sparse_reduce_batch(s["in_idx"], s["in_val"], s["off"], s["lo_hi"], c["B"], c["P"],
                                    c["width"], s["idx"], s["val"], s["cap"], s["nnz"], s["ws"])
        return {"idx": s["idx"], "val": s["val"], "nnz": s["nnz"]}

    grad, residual = _next_grad(s), s["residual"]
    out = {"residual": residual, "idx": s["idx"], "val": s["val"], "nnz": s["nnz"]}
    if kind in ("refresh", "step"):
        okt.okt_accumulate_topk_select(grad, residual, LR, s["k"], s["th"], s["count"], s["idx"],
                                       s["val"], s["nnz"], s["ws"])
        out.update({"th": s["th"], "count": s["count"]})
    elif kind == "reuse":
        okt.okt_accumulate_select(grad, residual, LR, s["th"], s["idx"], s["val"], s["nnz"], s["ws"])
    elif kind == "separate":
        okt.okt_residual_accumulate(grad, residual, LR)
        okt.okt_topk_threshold_exact(residual, s["k"], s["th"], s["count"], s["ws"])
        okt.okt_threshold_select(residual, s["th"], s["idx"], s["val"], s["nnz"], s["ws"])
        out.update({"th": s["th"], "count": s["count"]})
    elif kind == "literal":
        okt.okt_residual_accumulate(grad, residual, LR)
        okt.okt_threshold_select_copy(residual, s["th"], s["idx"], s["val"], s["nnz"], s["ws"])
        okt.okt_topk_threshold_exact(s["red_val"], s["k_global"], s["gth"], s["gcount"], s["ws"])
        okt.okt_coo_threshold_select(s["red_idx"], s["red_val"], s["red_nnz"], s["gth"], s["gidx"],
                                     s["gval"], s["gnnz"], s["ws"])
        okt.okt_index_intersect_zero(residual, s["idx"], s["nnz"], s["all_idx"], s["all_nnz"],
                                     s["ncommon"], s["ws"], indexes_out=s["common"])
    if kind == "step":
        okt.okt_region_partition(s["idx"], s["nnz"], s["n"], s["R"], s["bounds"], s["offsets"])
        r = s["reduce"]
        okt.okt_sparse_reduce(r["in_idx"], r["in_val"], r["off"], r["lo"], r["hi"], r["idx"],
                              r["val"], r["nnz"], r["ws"])
        okt.okt_topk_threshold_exact(r["val"], s["k_global"], s["gth"], s["gcount"], s["ws"])
        okt.okt_coo_threshold_select(r["idx"], r["val"], r["nnz"], s["gth"], s["gidx"], s["gval"],
                                     s["gnnz"], s["ws"])
        okt.okt_index_intersect_restore(residual, s["idx"], s["val"], s["nnz"], s["all_idx"],
                                        s["all_nnz"], s["ncommon"], s["ws"], indexes_out=s["common"])
        out.update({"bounds": s["bounds"], "offsets": s["offsets"], "red_idx": r["idx"],
                    "red_val": r["val"], "red_nnz": r["nnz"]})
    if kind in ("step", "literal"):
        out.update({"gth": s["gth"], "gcount": s["gcount"], "gidx": s["gidx"], "gval": s["gval"],
                    "gnnz": s["gnnz"], "common": s["common"], "ncommon": s["ncommon"]})
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without, and how exact it is
# ---------------------------------------------------------------------------
def _reduce_work(case, regions):
    e, u = _entries_expected(case) * regions, _union(case) * regions
    dense = 4 * case["width"] if case["kind"] == "region" else 0
    return {"bytes": 8 * e + 8 * u + dense, "flops": e}


def work(case):
    kind = case["kind"]
    if kind in ("region", "batch"):
        return _reduce_work(case, case.get("B", 1))
    n, k = case["n"], _k(case)
    read_both_write, select = 12 * n, 8 * k
    if kind in ("refresh", "reuse"):
        return {"bytes": read_both_write + select, "flops": 2 * n}
    if kind == "separate":                    # the threshold and the select each read the vector
        return {"bytes": read_both_write + 4 * n + 4 * n + 12 * k, "flops": 2 * n}
    # the global stage: the reduced values twice, what is selected of them, both index
    # lists, the intersection and the residual at its places
    reduced = _union(_own_region(case)) if kind == "step" else k
    stage = 4 * reduced + 4 * reduced + 12 * (reduced / 3) + 4 * k + 6 * k + 8 * (k / 2)
    if kind == "literal":
        return {"bytes": read_both_write + 4 * n + select + stage, "flops": 2 * n}
    r = _reduce_work(_own_region(case), 1)
    return {"bytes": read_both_write + select + r["bytes"] - 4 * _own_region(case)["width"] + stage,
            "flops": 2 * n + r["flops"]}


def tolerance(case):
    # The dense part and the global stage round as two fp32 operations do and otherwise
    # copy and count: the same bits.  The reduce sums in fp64 in any order and rounds once
    # to fp32: it stands 2.5e-8 (2-norm) and at most 6e-8 of a value off the exact sum;
    # four times that.
    if case["kind"] in ("region", "batch", "step"):
        return {"rel": 1e-7, "max": 2.4e-7}
    return "exact"


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
def _at_front(values, size):
    out = torch.zeros(size, dtype=torch.float64, device=DEV)
    out[:values.numel()] = values[:size]
    return out


def _exact_reduce(s, lo, width):
    """Sums of one region's entries in 64 bits: (dense, hit)."""
    at = s["in_idx"].long() - lo
    dense = torch.zeros(width, dtype=torch.float64, device=DEV)
    dense.index_add_(0, at, s["in_val"].double())
    hit = torch.zeros(width, dtype=torch.bool, device=DEV)
    hit[at] = True
    return dense, hit


def exact(case, seed):
    kind = case["kind"]
    s = prepare(case, seed)
    if kind == "region":
        dense, hit = _exact_reduce(s, s["lo"], case["width"])
        return {"idx": None, "val": _at_front(dense[hit], s["val"].numel()), "nnz": None,
                "dense": dense}
    if kind == "batch":
        B, P, width = case["B"], case["P"], case["width"]
        val = torch.zeros(B * s["cap"], dtype=torch.float64, device=DEV)
        lo = s["lo_hi"][::2].tolist()
        off = s["off"].reshape(B, P + 1)[:, [0, P]].tolist()
        for b in range(B):
            part = {k: s[k][off[b][0]:off[b][1]] for k in ("in_idx", "in_val")}
            dense, hit = _exact_reduce(part, lo[b], width)
            sums = dense[hit][:s["cap"]]
            val[b * s["cap"]:b * s["cap"] + sums.numel()] = sums
        return {"idx": None, "val": val, "nnz": None}
    grad, residual = s["ring"][0], s["residual"]
    acc = _accumulate(residual, grad)                  # decides what is selected, in fp32
    mag = acc.abs()
    th = s["th"] if kind in ("reuse", "literal") else _kth_largest(mag, s["k"])
    chosen = mag >= th
    wide = residual.double().add_(grad.double().mul_(float(np.float32(LR))))
    picked = wide[chosen]
    out = {"idx": None, "nnz": None, "val": _at_front(picked, s["val"].numel())}
    if kind in ("refresh", "separate", "step"):
        out.update({"th": picked.abs().min().reshape(1), "count": None})
    if kind in ("refresh", "reuse", "separate"):
        out["residual"] = wide.masked_fill_(chosen, 0.0)
        return out
    everywhere = torch.zeros(s["n"], dtype=torch.bool, device=DEV)
    everywhere[s["all_idx"].long()] = True
    out["residual"] = wide.masked_fill_(chosen & everywhere, 0.0)
    if kind == "step":
        r = s["reduce"]
        dense, hit = _exact_reduce(r, r["lo"], r["hi"] - r["lo"])
        red = dense[hit]
        full = _at_front(red, r["val"].numel())
        out.update({"bounds": None, "offsets": None, "red_idx": None, "red_val": full,
                    "red_nnz": None})
    else:
        full = s["red_val"].double()
        red = full[:int(s["red_nnz"])]
    gth = full.abs().sort(descending=True).values[s["k_global"] - 1]
    out.update({"gth": gth.reshape(1), "gcount": None, "gidx": None,
                "gval": _at_front(red[red.float().abs() >= gth.float()], s["gval"].numel()),
                "gnnz": None, "common": None, "ncommon": None})
    return out
