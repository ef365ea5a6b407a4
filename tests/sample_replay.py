"""Host replay of the exact threshold's sample, for tests that have to know which path a
vector takes: which elements the sample reads, the bound it finds, and what the call left
in its workspace about it."""
import numpy as np

RUN, RUNS, WORKGROUPS = 16, 8192, 16       # elements a run, runs, workgroups (run r: workgroup r mod 16)
SHIFT = 18                                 # the key's 13 highest bits are the bin


def key_of(x):
    return np.ascontiguousarray(x, dtype=np.float32).view(np.uint32) & np.uint32(0x7FFFFFFF)


def run_starts(n):
    """First element of each of the sampled runs."""
    return np.arange(RUNS, dtype=np.uint64) * np.uint64(n // RUN) // np.uint64(RUNS) * np.uint64(RUN)


def sampled(n):
    """True where the sample reads a vector of n elements."""
    mask = np.zeros(n, dtype=bool)
    for j in range(RUN):
        mask[run_starts(n).astype(np.int64) + j] = True
    return mask


def bounds(n, k, positions, keys):
    """The workgroups' bounds for a vector of n elements whose keys are `keys` at the
    (distinct) `positions` and zero elsewhere.  The least of them is the one in force."""
    starts = run_starts(n)
    per_wg = RUNS // WORKGROUPS * RUN
    kp = (k * per_wg + n // 2) // n
    rank = min(max(kp + int(np.float32(np.sqrt(np.float32(kp))) + np.float32(0.5)), 1), per_wg)
    # a vector shorter than the sample has runs that are read more than once
    run, times = np.unique(starts, return_counts=True)
    first = np.concatenate([[0], np.cumsum(times)[:-1]])
    pos, keys = np.asarray(positions, dtype=np.uint64), np.asarray(keys, dtype=np.uint32)
    at = np.searchsorted(run, pos, side="right").astype(np.int64) - 1
    inside = pos - run[at] < RUN
    seen = [[] for _ in range(WORKGROUPS)]
    for a, key in zip(at[inside], keys[inside]):
        for r in range(first[a], first[a] + times[a]):
            seen[r % WORKGROUPS].append(int(key))
    out = []
    for s in seen:
        s.sort(reverse=True)
        out.append((s[rank - 1] if len(s) >= rank else 0) >> SHIFT << SHIFT)
    return np.array(out, dtype=np.uint32)


def bounds_dense(acc, k):
    """The same for a vector given in full."""
    mask = sampled(acc.size)
    return bounds(acc.size, k, np.flatnonzero(mask), key_of(acc[mask]))


class State:
    """What a call left at the start of its workspace: the bounds, the candidates found by
    okt_topk_threshold_exact and by okt_accumulate_topk_select."""

    def __init__(self, ws):
        raw = ws[:96].cpu().numpy()
        self.bounds = raw[:64].view(np.uint32)
        self.keys_found = int(raw[64:72].view(np.uint64)[0])
        self.collected = int(raw[80:88].view(np.uint64)[0])
