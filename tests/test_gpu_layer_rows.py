"""GPU tests of layers just above the size every layer is a row at, split into parts
whose select workgroup holds the whole selection interval (the default rule;
row_max is not set here), against the oracle, bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from _gpu_common import log, same_bits, torch_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sc():
    import paper_2301_08897_amd as m
    return m


# interval around the k-th key: narrow, wide (as much as fits), and full of ties;
# the last layer is one element past the longest that is a row
@pytest.mark.parametrize("ratio,kind", [(0.01, "normal"), (0.1, "laplace"), (0.05, "ties"), (0.001, "normal")])
def test_long_rows(sc, ratio, kind):
    log(f"layer rows: ratio {ratio}, {kind}")
    torch, dev = torch_dev()
    sizes = [2**21 + 1, 70_001, 2**22 if kind == "normal" else 3_000_003, 300, 2**22 + 1]
    seg_off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n, K = int(seg_off[-1]), 2
    rng = np.random.default_rng(int(ratio * 1000))
    room = torch.zeros(K, n + 1, dtype=torch.float32, device=dev)      # rows at different 4-byte offsets
    G = np.empty((K, n), dtype=np.float32)
    for j in range(K):
        x = rng.laplace(size=n) if kind == "laplace" else rng.standard_normal(n)
        if kind == "ties":
            x = np.sign(x) * np.floor(np.abs(x) * 256) / 256
        G[j] = x.astype(np.float32)
        room[j, j:j + n].copy_(torch.from_numpy(G[j]))
    sel = sc.LayerSelect([room[j, j:j + n] for j in range(K)], seg_off, [ratio] * K)
    idx, val, _ = sel.run()
    torch.cuda.synchronize()
    for j in range(K):
        ref = [oracle.topk_by_threshold(G[j, a:b], oracle.topk_k(b - a, ratio)) for a, b in
               zip(seg_off[:-1], seg_off[1:])]
        want = np.concatenate([r[0].astype(np.int64) + a for r, a in zip(ref, seg_off[:-1])]).astype(np.uint32)
        assert np.array_equal(idx[j].cpu().numpy(), want), f"device {j}: indices"
        assert same_bits(val[j].cpu().numpy(), G[j][want]), f"device {j}: values"
