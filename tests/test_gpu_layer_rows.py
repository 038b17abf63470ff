"""GPU tests of layers just above the size every layer is a row at (the default
rule, row_max -1) and of split rows whose values do not spread as a sample's would,
against the oracle, bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from _gpu_common import check_energies, log, same_bits, torch_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sc():
    import paper_2301_08897_amd as m
    m.set_option("row_max", -1)
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


# Rows whose values do not spread as a random sample's would: equal keys that no
# bracket tells apart, within and beyond what the candidate list holds; kept
# entries in one run; mostly zeros; values that the sampled positions (256 of
# every 4096) miss or are all of.
KINDS = ("ties", "flood", "clusters", "zeros", "miss", "peak")
SIZES = (2**21 + 5, 70_001, 300_003, 5_000, 16384 * 5 - 2)


def uneven(rng, kind, n, ratio):
    x = rng.standard_normal(n).astype(np.float32)
    sign = np.where(rng.random(n) < 0.5, np.float32(-1), np.float32(1))
    at = np.arange(n)
    if kind in ("ties", "flood"):             # 2.5% (more keys than LDS holds in the longest row) and 25%
        m = np.quantile(np.abs(x), 1.0 - ratio / 2).astype(np.float32)       # inside the kept set
        x = np.where(rng.random(n) < (0.025 if kind == "ties" else 0.25), sign * m, x)
    elif kind == "clusters":
        x[n // 3:n // 3 + n // 24] *= np.float32(50)
    elif kind == "zeros":
        x *= rng.random(n) < 0.004
    else:
        x *= np.where((at % 4096 < 260) == (kind == "peak"), np.float32(1), np.float32(0.01))
    return x.astype(np.float32)


# (the last set: split rows short enough for a workgroup each when they are slow)
@pytest.mark.parametrize("ratio", [0.02, 0.001])
@pytest.mark.parametrize("kinds,sizes", [((k,) * 2, SIZES) for k in KINDS] + [(KINDS + ("normal",), SIZES)]
                         + [(KINDS + ("normal",), (200_001,) + SIZES[3:])])
def test_uneven_rows(sc, ratio, kinds, sizes):
    log(f"uneven layer rows: ratio {ratio}, {kinds}, {len(sizes)} layers")
    torch, dev = torch_dev()
    seg_off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n, K = int(seg_off[-1]), len(kinds)
    rng = np.random.default_rng(K)
    room = torch.zeros(K, n + 4, dtype=torch.float32, device=dev)
    G = np.empty((K, n), dtype=np.float32)
    for j, kind in enumerate(kinds):
        G[j] = np.concatenate([uneven(rng, kind, m, ratio) if kind != "normal" else
                               rng.standard_normal(m).astype(np.float32) for m in sizes])
        room[j, j % 4:j % 4 + n].copy_(torch.from_numpy(G[j]))
    sel = sc.LayerSelect([room[j, j % 4:j % 4 + n] for j in range(K)], seg_off, [ratio] * K)
    for again in range(2):                    # the second call finds the first one's workspace
        for t in sel.idx + sel.val:
            t.view(torch.int32).fill_(-1)
        idx, val, en = sel.run()
        torch.cuda.synchronize()
        e = en.cpu().numpy()
        for j in range(K):
            want = np.concatenate([oracle.topk_by_threshold(G[j, a:b], oracle.topk_k(b - a, ratio))[0].astype(np.int64) + a
                                   for a, b in zip(seg_off[:-1], seg_off[1:])]).astype(np.uint32)
            assert np.array_equal(idx[j].cpu().numpy(), want), f"call {again}, device {j} ({kinds[j]}): indices"
            assert same_bits(val[j].cpu().numpy(), G[j][want]), f"call {again}, device {j} ({kinds[j]}): values"
            check_energies(f"device {j}", e[2 * j], e[2 * j + 1], oracle.energies_extended(G[j], want), n, want.size)


def test_many_slow_rows(sc):
    """More slow rows than a wave looks over at once, beside others that are not."""
    log("many slow layer rows")
    torch, dev = torch_dev()
    sizes, K, ratio = (66_001, 70_003, 900), 40, 0.01
    seg_off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(seg_off[-1])
    rng = np.random.default_rng(40)
    G = np.stack([np.concatenate([uneven(rng, "zeros" if j % 5 else "clusters", m, ratio) for m in sizes])
                  for j in range(K)])
    idx, val, _ = sc.LayerSelect(torch.from_numpy(G).to(dev), seg_off, [ratio] * K).run()
    torch.cuda.synchronize()
    for j in range(K):
        want = np.concatenate([oracle.topk_by_threshold(G[j, a:b], oracle.topk_k(b - a, ratio))[0].astype(np.int64) + a
                               for a, b in zip(seg_off[:-1], seg_off[1:])]).astype(np.uint32)
        assert np.array_equal(idx[j].cpu().numpy(), want), f"device {j}: indices"
        assert same_bits(val[j].cpu().numpy(), G[j][want]), f"device {j}: values"
