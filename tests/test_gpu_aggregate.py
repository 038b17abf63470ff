"""GPU tests of the aggregation's dense contributions against the oracle, bit
for bit: range remainders, gradients at every 4-byte offset, dense devices at
the ends and in a row, and a device that turns dense although the rule always
sends Top-k."""
from __future__ import annotations

import math

import numpy as np
import pytest

import oracle
from _gpu_common import log, same_bits, torch_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sc():
    import paper_2301_08897_amd as m
    return m


# ranges are 2048 positions: a lone short one, whole ones, a remainder of one, two, three
@pytest.mark.parametrize("n", [1, 3, 127, 2047, 2048, 2049, 4098, 6147, 100_003])
@pytest.mark.parametrize("dense", [(0,), (2, 3, 5), (0, 1, 2, 3, 4, 5, 6, 7, 8), (8,)])
def test_dense_contributions(sc, n, dense):
    log(f"aggregate dense n={n} dense={dense}")
    torch, dev = torch_dev()
    rng = np.random.default_rng(n + len(dense))
    K = 9
    sets, dsets = [], []
    for j in range(K):
        if j in dense:
            v = rng.standard_normal(n).astype(np.float32)
            room = torch.zeros(n + 4, dtype=torch.float32, device=dev)
            d = room[j % 4:j % 4 + n]
            d.copy_(torch.from_numpy(v))
            sets.append((None, v))
            dsets.append((None, d))
        else:
            k = int(rng.integers(0, n + 1))
            idx = np.sort(rng.choice(n, size=k, replace=False)).astype(np.uint32)
            v = rng.standard_normal(k).astype(np.float32)
            sets.append((idx, v))
            dsets.append((torch.from_numpy(idx).to(dev), torch.from_numpy(v).to(dev)))
    w = rng.random(K)
    w = (w / w.sum()).astype(np.float32)
    got = sc.weighted_aggregate(dsets, w, n)
    torch.cuda.synchronize()
    assert same_bits(got.cpu().numpy(), oracle.aggregate(sets, w, n))


@pytest.mark.parametrize("momentum", [False, True])
def test_dense_although_always_compressing(sc, momentum):
    """With delta = +inf a device sends its dense gradient only when its energies are
    not finite; its values then still reach the aggregate and the update."""
    log(f"aggregate device with an infinite entry, momentum={momentum}")
    torch, dev = torch_dev()
    rng = np.random.default_rng(3)
    K, n, ratio = 3, 70_003, 0.01
    G = rng.standard_normal((K, n)).astype(np.float32)
    G[1, 5] = np.inf
    p = rng.standard_normal(n).astype(np.float32)
    g_dev, p_dev = torch.from_numpy(G).to(dev), torch.from_numpy(p).to(dev)
    more = {}
    if momentum:
        more = dict(momentum_buf=torch.zeros(n, dtype=torch.float32, device=dev), momentum=0.9, weight_decay=1e-4)
    step = sc.FusedStep(g_dev, [ratio] * K, delta=math.inf, params=p_dev, **more)
    w = np.array([0.5, 0.25, 0.25], dtype=np.float32)
    out = step.run(w, 0.1)
    torch.cuda.synchronize()
    assert out.compressed.cpu().numpy().tolist() == [1, 0, 1]
    sets = [(None, G[j]) if j == 1 else oracle.topk(G[j], oracle.topk_k(n, ratio))[:2] for j in range(K)]
    with np.errstate(invalid="ignore"):
        dense = oracle.aggregate(sets, w, n)
    assert np.isinf(dense[5]) and same_bits(out.dense.cpu().numpy(), dense)
    if momentum:
        p_ref, v_ref = oracle.momentum_sgd(p, np.zeros_like(p), dense, 0.1, 0.9, 1e-4)
        assert same_bits(step.momentum_buf.cpu().numpy(), v_ref)
    else:
        p_ref = oracle.sgd(p, dense, 0.1)
    assert same_bits(p_dev.cpu().numpy(), p_ref)
