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
    kept = [oracle.topk_by_threshold(G[j], oracle.topk_k(n, ratio))[0] for j in range(K)]
    sets = [(i, G[j][i]) for j, i in enumerate(kept)]
    for j in range(K):
        assert np.array_equal(out.idx[j].cpu().numpy(), sets[j][0]), f"device {j}: indices"
        assert same_bits(out.val[j].cpu().numpy(), sets[j][1]), f"device {j}: values"
    assert same_bits(out.dense.cpu().numpy(), oracle.aggregate(sets, w, n))


# ties from just before, at and just after a tile's and a chunk's start, for less
# than a window, a chunk and more than a tile
RUNS = [(0, 700), (3 * TILE - 5, 30_000), (2 * TILE + CHUNK + 1, 3 * CHUNK), (5 * TILE, TILE),
        (12 * TILE - 700, 703)]


def tied(K, n, shift, start, length):
    rng = np.random.default_rng(start + shift)
    G = (rng.standard_normal((K, n), dtype=np.float32) * np.float32(0.01)).astype(np.float32)
    sign = rng.choice(np.array([-1.0, 1.0], dtype=np.float32), size=(K, length))
    G[:, start:start + length] = sign * np.float32(0.25)
    G[1::2, ::97] = np.float32(3.0)            # keys above the tied ones in every tile
    return G


# 2 devices of 13 tiles take the output's 1024-thread workgroups, 41 (more than 512
# tiles in all) its 512-thread ones
@pytest.mark.parametrize("K,shift", [(2, 0), (2, 1), (2, 3), (41, 1), (41, 3)])
@pytest.mark.parametrize("start,length", RUNS)
def test_tied_run(sc, K, shift, start, length):
    log(f"hot tiles: {K} devices, {length} ties from {start}, offset {shift}")
    fused(sc, tied(K, 12 * TILE + 3, shift, start, length), 0.02, shift)


# more than 1024 tiles per device: offsets from a launch of their own, for 512-thread
# workgroups and, with more than 16384 tiles in all, 256-thread ones
@pytest.mark.parametrize("K,shift", [(1, 1), (1, 3), (16, 3)])
def test_tied_run_of_many_tiles(sc, K, shift):
    log(f"hot tiles: {K} devices of 1025 tiles, offset {shift}")
    n = 1024 * TILE + 3
    G = tied(K, n, shift, 1000 * TILE - 5, 30_000)
    G[:, 1024 * TILE - 700:] = np.float32(-0.25)              # the last, partial tile too
    G[:, :900] = np.float32(0.25)
    fused(sc, G, 0.002, shift)


# a long layer's output, with 256-thread workgroups
@pytest.mark.parametrize("shift", [1, 3])
@pytest.mark.parametrize("start,length", RUNS)
def test_tied_run_of_a_layer(sc, shift, start, length):
    log(f"hot tiles: a layer, {length} ties from {start}, offset {shift}")
    torch, dev = torch_dev()
    K, n, ratio = 2, 12 * TILE + 3, 0.02
    G = tied(K, n, shift, start, length)
    room = torch.zeros(K, n + 8, dtype=torch.float32, device=dev)
    grads = []
    for j in range(K):
        base = (-room[j].data_ptr() // 4) % 4 + shift
        grads.append(room[j][base:base + n])
        grads[j].copy_(torch.from_numpy(G[j]))
    sc.set_option("row_max", 0)
    try:
        idx, val, _ = sc.LayerSelect(grads, [0, n], [ratio] * K).run()
        torch.cuda.synchronize()
    finally:
        sc.set_option("row_max", -1)
    for j in range(K):
        want = oracle.topk_by_threshold(G[j], oracle.topk_k(n, ratio))[0]
        assert np.array_equal(idx[j].cpu().numpy(), want), f"device {j}: indices"
        assert same_bits(val[j].cpu().numpy(), G[j][want]), f"device {j}: values"


def test_interval_keys_overflow_one_segment(sc):
    """Every second tile all ties: the interval keys of the hot tiles overrun their
    list segment, and the device takes the exact path."""
    log("hot tiles: list segment overflow")
    n, ratio = 128 * TILE + 5, 0.14
    # 129 tiles take two segments in turn, so the tied tiles' keys share one, which
    # holds as many as the device's whole list: 2 k + n / 8
    k = oracle.topk_k(n, ratio)
    assert 64 * TILE > 2 * k + n // 8 + 128 and 2 * (2 * k + n // 8 + 64) <= n
    rng = np.random.default_rng(5)
    G = (rng.standard_normal((2, n)) * 0.01).astype(np.float32)
    for t in range(0, 128, 2):
        G[0, t * TILE:(t + 1) * TILE] = np.float32(-0.5)
    fused(sc, G, ratio, 0)
