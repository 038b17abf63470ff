"""GPU test that a device's energies are the same bits however its call is
launched: alone or with other devices, in 1 to 4 device groups, as a layer of
its own. These runs differ in the output's workgroup size (256, 512 or 1024
threads, by the number of tiles), which must not change the order of the sums."""
from __future__ import annotations

import numpy as np
import pytest

from _gpu_common import log, same_bits, torch_dev

pytestmark = pytest.mark.gpu

K, N, RATIO, BETA = 4, 2_500_003, 0.02, 0.9     # 153 tiles per device: 612 in one group, 306 in two


@pytest.fixture(scope="module")
def sc():
    import paper_2301_08897_amd as m
    return m


# the exact path (all tiles read again for the output), and hot tiles only; few
# tiles hold the kept entries, so that a tile's last bits show in the device's sum
@pytest.mark.parametrize("path", ["force_exact", "hot"])
def test_energy_bits_independent_of_launch(sc, path):
    log(f"energy order: {path}")
    torch, dev = torch_dev()
    rng = np.random.default_rng(8)
    G = (rng.standard_normal((K, N)) * 0.01).astype(np.float32)
    G[:, 700_001:760_000] *= np.float32(300.0)
    g = torch.from_numpy(G).to(dev)
    w = np.full(K, 1.0 / K, dtype=np.float32)
    ref = {}

    def same(what, got, key):
        got = got.cpu().numpy()
        first = ref.setdefault(key, got)
        assert same_bits(got.view(np.uint32), first.view(np.uint32)), f"{what}: {key} differs"

    if path == "force_exact":
        sc.set_option("force_exact", 1)
    try:
        for parts in (1, 2, 3, 4):
            sc.set_option("parts", parts)
            step = sc.FusedStep(g, [RATIO] * K, delta=0.9, ewma_beta=BETA)
            for it in range(2):
                step.run(w)
                torch.cuda.synchronize()
                same(f"parts {parts}", step.energies, "energies")
                same(f"parts {parts}", step.ewma, f"moving averages of iteration {it}")
        sc.set_option("parts", 1)
        for j in range(K):
            _, _, en = sc.topk_select(g[j], RATIO, energies=True)
            torch.cuda.synchronize()
            assert same_bits(en.cpu().numpy().view(np.uint32), ref["energies"][2 * j:2 * j + 2].view(np.uint32)), \
                f"device {j} alone"
        sc.set_option("row_max", 0)
        sel = sc.LayerSelect(g, [0, N], [RATIO] * K)
        sel.run()
        torch.cuda.synchronize()
        same("a layer of its own", sel.energies, "energies")
    finally:
        sc.set_option("row_max", -1)
        sc.set_option("parts", 1)
        sc.set_option("force_exact", 0)
