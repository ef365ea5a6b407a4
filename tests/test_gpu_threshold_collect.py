"""The pass that collects the candidates of the exact threshold deals a workgroup's elements out
to its waves: lengths around whole rounds, batches and workgroups, with the answer in the last
elements of the vector, where a round that is left out would show."""
import numpy as np
import pytest
import torch

import paper_2201_07598_amd as okt
from oracle import okt_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("base", [65_792, 16 * 1024 * 7, 262_144, 3_000_064, 4_194_304, 8_388_608 + 16_384])
@pytest.mark.parametrize("off", [-1025, -257, -256, -1, 0, 1, 3, 255, 256, 257, 1023, 1024, 1025, 4097, 15_361])
def test_every_element_is_seen(base, off):
    n = max(base + off, 65_537)
    k = 2_000
    rng = np.random.default_rng(n)
    acc = (rng.standard_normal(n) * 1e-3).astype(np.float32)
    acc[-k // 2:] = np.linspace(1.0, 2.0, k // 2, dtype=np.float32)       # the largest lie at the end,
    acc[: k // 2 - 1] = -3.0                                             # and at the front
    th = torch.zeros(1, device=DEV)
    count = torch.zeros(1, dtype=torch.int64, device=DEV)
    ws = torch.empty(okt.okt_workspace_bytes(n, 1), dtype=torch.uint8, device=DEV)
    okt.okt_topk_threshold_exact(torch.from_numpy(acc).to(DEV), k, th, count, ws)
    want = orc.topk_threshold_exact(acc, k)
    want_th, want_count = (want["threshold"], want["count_ge"]) if isinstance(want, dict) else want
    assert float(th) == float(want_th) and int(count) == int(want_count)
