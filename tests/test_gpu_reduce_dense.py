"""Dense tiles of the reduce: their hits leave through LDS in output order.  Regions that end at,
before and behind the edges of tiles and of bitmap words, all slots hit, hardly any, outputs cut
short inside a tile, the dense copy.  Sums of dyadic values: exact in any order."""
import numpy as np
import pytest
import torch

import paper_2201_07598_amd as okt
from oracle import okt_oracle as orc
from test_gpu_reduce_tiles import DEV, dev, run_batch, some

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [1, 31, 32, 33, 4_095, 4_096, 4_097, 9_215, 9_216, 9_217, 18_433])
@pytest.mark.parametrize("B,P", [(3, 2), (530, 2), (530, 70)])
def test_edges_of_dense_tiles(B, P, width):
    rng = np.random.default_rng(width + B + P)
    full = np.arange(width, dtype=np.uint32)
    regions = []
    for b in range(B):
        lo = 5 * b
        if b in (0, B - 1):
            ps = [full + np.uint32(lo)] + [some(rng, lo, width, max(1, width // 3)) for _ in range(P - 1)]
        elif b == 1:
            ps = [some(rng, lo, width, 1) for _ in range(P)]
        else:
            ps = [np.array([lo + width - 1], np.uint32)] * P
        regions.append((lo, lo + width, ps))
    run_batch(regions, P, width, width, lead=1)
    run_batch(regions, P, width, max(1, (2 * width) // 3))       # cut short (two contributions take ranked tiles then)
    run_batch(regions, P, width, max(1, width - width // 20))    # cut short in dense ones


@pytest.mark.parametrize("width", [9_215, 9_216, 9_217, 18_433])
def test_dense_copy_of_wide_dense_tiles(width):
    """Tiles of 9,216 slots, in a launch of enough of them."""
    rng = np.random.default_rng(width)
    B, P = 530, 70
    regions = []
    for b in range(B):
        ps = [some(rng, 3 * b, width, width // 2) if b in (0, B - 1) else np.array([3 * b + p], np.uint32) for p in range(P)]
        regions.append((3 * b, 3 * b + width, ps))
    run_batch(regions, P, width, width, lead=3, dense=True)
    run_batch(regions, P, width, width // 2, dense=True)         # sparse outputs cut short, dense ones whole


@pytest.mark.parametrize("width", [33, 4_097, 9_217])
def test_dense_copy_of_dense_tiles(width):
    """One region: tiles of 4,096 slots."""
    rng = np.random.default_rng(width)
    lo, P = 77, 3
    ps = [some(rng, lo, width, width // 2) for _ in range(P)]
    idx = np.concatenate(ps)
    val = (rng.integers(-2048, 2048, idx.size) * 2.0 ** -12).astype(np.float32)
    off = np.concatenate([[0], np.cumsum([p.size for p in ps])]).astype(np.uint64)
    ref = orc.sparse_reduce(idx, val, off, lo, lo + width)
    o_idx = torch.zeros(width, dtype=torch.int32, device=DEV)
    o_val, dense = torch.zeros(width, device=DEV), torch.full((width,), 7.0, device=DEV)
    nnz = torch.zeros(2, dtype=torch.int64, device=DEV)
    ws = torch.empty(okt.okt_sparse_reduce_batch_workspace_bytes(1, P, width), dtype=torch.uint8, device=DEV)
    okt.okt_sparse_reduce(dev(idx), dev(val), dev(off), lo, lo + width, o_idx, o_val, nnz, ws, dense_out=dense)
    torch.cuda.synchronize()
    U = ref["idx"].size
    assert nnz.tolist() == [U, U]
    want = ref["val"].astype(np.float32)
    assert np.array_equal(o_idx.cpu().numpy().view(np.uint32)[:U], ref["idx"])
    assert np.array_equal(o_val.cpu().numpy()[:U], want)
    full = np.zeros(width, np.float32)
    full[ref["idx"].astype(np.int64) - lo] = want
    assert np.array_equal(dense.cpu().numpy(), full)
