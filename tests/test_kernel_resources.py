"""CPU test of the registers that the output kernels were compiled to, from the
metadata of the built library: their staged tiles are bound by latency, so the
launches without own offsets need eight waves per SIMD (512 vector registers: at
most 64 each), and none may spill."""
from __future__ import annotations

import os
import re
import shutil
import subprocess

LLVM = "/opt/rocm/llvm/bin"


def kernels(tmp_path):
    """Name -> {vgpr_count, vgpr_spill_count, private_segment_fixed_size} of every kernel."""
    from paper_2301_08897_amd import LIB_PATH
    lib = shutil.copy(LIB_PATH, tmp_path)
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    found = {}
    for f in os.listdir(tmp_path):
        if "gfx950" not in f:
            continue
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", f], cwd=tmp_path, check=True, capture_output=True,
                               text=True).stdout
        name = None
        for key, value in re.findall(r"^\s+\.(\w+):\s+(\S+)$", notes, re.M):
            if key == "name" and value.startswith("_ZN7scadles"):
                name = value
                found[name] = {}
            elif name and key in ("vgpr_count", "vgpr_spill_count", "private_segment_fixed_size"):
                found[name].setdefault(key, int(value))
    return found


def test_output_kernels_registers(tmp_path):
    writes = {k: v for k, v in kernels(tmp_path).items() if "7k_writeI" in k}
    assert len(writes) == 4, sorted(writes)
    for name, r in writes.items():
        assert r["vgpr_spill_count"] == 0 and r["private_segment_fixed_size"] == 0, (name, r)
        own_offsets = "Lb1E" in name
        assert r["vgpr_count"] <= (72 if own_offsets else 64), (name, r)
