"""GPU tests of tiles with more candidates than their slot holds, against the
oracle, bit for bit: runs of tied magnitudes across tile and chunk edges, at every
4-byte offset of the gradient, and interval keys that overflow their list."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from _gpu_common import log, same_bits, torch_dev

pytestmark = pytest.mark.gpu

TILE, CHUNK = 16384, 4096


@pytest.fixture(scope="module")
def sc():
    import paper_2301_08897_amd as m
    return m


def fused(sc, G, ratio, shift):
    """One fused step over devices whose gradients start at a 4-byte offset of `shift`."""
    torch, dev = torch_dev()
    K, n = G.shape
    room = torch.zeros(K, n + 8, dtype=torch.float32, device=dev)
    grads = []
    for j in range(K):
        flat = room[j]
        base = (-flat.data_ptr() // 4) % 4
        g = flat[base + shift:base + shift + n]
        g.copy_(torch.from_numpy(G[j]))
        assert g.data_ptr() // 4 % 4 == shift
        grads.append(g)
    step = sc.FusedStep(grads, [ratio] * K)
    w = np.full(K, 1.0 / K, dtype=np.float32)
    out = step.run(w)
    torch.cuda.synchronize()
    sets = [oracle.topk(G[j], oracle.topk_k(n, ratio))[:2] for j in range(K)]
    for j in range(K):
        assert np.array_equal(out.idx[j].cpu().numpy(), sets[j][0]), f"device {j}: indices"
        assert same_bits(out.val[j].cpu().numpy(), sets[j][1]), f"device {j}: values"
    assert same_bits(out.dense.cpu().numpy(), oracle.aggregate(sets, w, n))


# ties from just before, at and just after a tile's and a chunk's start, for less
# than a window, a chunk and more than a tile
@pytest.mark.parametrize("shift", [0, 1, 3])
@pytest.mark.parametrize("start,length", [(0, 700), (3 * TILE - 5, 30_000), (2 * TILE + CHUNK + 1, 3 * CHUNK),
                                          (5 * TILE, TILE), (12 * TILE - 700, 703)])
def test_tied_run(sc, shift, start, length):
    log(f"hot tiles: {length} ties from {start}, offset {shift}")
    n = 12 * TILE + 3
    rng = np.random.default_rng(start + shift)
    G = (rng.standard_normal((2, n)) * 0.01).astype(np.float32)
    sign = rng.choice(np.array([-1.0, 1.0], dtype=np.float32), size=(2, length))
    G[:, start:start + length] = sign * np.float32(0.25)
    G[1, ::97] = np.float32(3.0)               # keys above the tied ones in every tile
    fused(sc, G, 0.02, shift)


def test_interval_keys_overflow_one_segment(sc):
    """Every second tile all ties: the interval keys of the hot tiles overrun their
    list segment, and the device takes the exact path."""
    log("hot tiles: list segment overflow")
    n = 128 * TILE + 5
    rng = np.random.default_rng(5)
    G = (rng.standard_normal((2, n)) * 0.01).astype(np.float32)
    for t in range(0, 128, 2):
        G[0, t * TILE:(t + 1) * TILE] = np.float32(-0.5)
    fused(sc, G, 0.14, 0)
