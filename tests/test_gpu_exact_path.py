"""GPU tests of the exact path's digit passes against the oracle, bit for bit, at
sizes where their blocks are whole (at least 128 blocks of 8192 elements) and just
below: values all different, mostly zeros and tied, which are counted in different
ways, at every 4-byte offset; devices on the exact path beside sampled ones."""
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


def values(rng, kind, n):
    x = rng.standard_normal(n).astype(np.float32)
    if kind == "zeros":                       # fewer nonzero values than entries kept
        x *= rng.random(n) < 0.1
    elif kind == "ties":                      # 37% of the elements share a key with 16 others of their wave
        x = np.where(rng.random(n) < 0.37, np.sign(x) * np.float32(0.5), x).astype(np.float32)
    elif kind == "runs":                      # ties and other values in turn, by blocks
        x[(np.arange(n) // 5000) % 2 == 0] = np.float32(-0.75)
    return x


# eight devices: 16 blocks each from n = 15 * 8192 - 2 on
@pytest.mark.parametrize("n", [15 * 8192 - 3, 15 * 8192 + 1, 16 * 8192 - 3, 63 * 8192 + 1])
@pytest.mark.parametrize("kind", ["normal", "zeros", "ties", "runs", "mixed"])
def test_exact_path(sc, n, kind):
    log(f"exact path n={n} {kind}")
    torch, dev = torch_dev()
    K = 8
    rng = np.random.default_rng(n)
    kinds = ["normal", "zeros", "ties", "runs"]
    G = np.stack([values(rng, kinds[j % 4] if kind == "mixed" else kind, n) for j in range(K)])
    # "mixed": every other device small enough a ratio for the sampled path
    ratios = [0.3 if kind != "mixed" or j % 2 else 0.01 for j in range(K)]
    room = torch.zeros(K, n + 8, dtype=torch.float32, device=dev)
    grads = []
    for j in range(K):
        base = (-room[j].data_ptr() // 4) % 4 + j % 4
        grads.append(room[j][base:base + n])
        grads[j].copy_(torch.from_numpy(G[j]))
    w = np.full(K, 1.0 / K, dtype=np.float32)
    out = sc.FusedStep(grads, ratios).run(w)
    torch.cuda.synchronize()
    sets = [oracle.topk_by_threshold(G[j], oracle.topk_k(n, ratios[j]))[0] for j in range(K)]
    for j in range(K):
        assert np.array_equal(out.idx[j].cpu().numpy(), sets[j]), f"device {j}: indices"
        assert same_bits(out.val[j].cpu().numpy(), G[j][sets[j]]), f"device {j}: values"
    assert same_bits(out.dense.cpu().numpy(), oracle.aggregate([(i, G[j][i]) for j, i in enumerate(sets)], w, n))
