"""Registers of the built kernels: no sweep keeps anything in scratch memory
(the built library's own metadata; no GPU)."""
import os
import re
import struct
import subprocess

import pytest

from paper_2609_33814_amd import bdrs

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


def kernels(tmp_path):
    """name -> metadata text of every gfx950 kernel in the library."""
    tools = [os.path.join(LLVM, t) for t in ("llvm-objcopy", "llvm-readelf")]
    if not all(os.path.exists(t) for t in tools):
        pytest.skip("LLVM tools not available")
    bdrs.lib()  # it has been built
    fat = tmp_path / "fatbin"
    subprocess.run([tools[0], "--dump-section", f".hip_fatbin={fat}", bdrs.LIB_PATH, os.devnull], check=True)
    data, found, at = fat.read_bytes(), {}, 0
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        (count,), pos = struct.unpack_from("<Q", data, at + 24), at + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + length].decode()
            pos += 24 + length
            if "gfx950" not in target or not size:
                continue
            obj = tmp_path / f"{at}.o"
            obj.write_bytes(data[at + offset:at + offset + size])
            notes = subprocess.run([tools[1], "--notes", str(obj)], check=True, capture_output=True, text=True).stdout
            for text in notes.split("  - .agpr_count")[1:]:
                found[re.search(r"\.name:\s+(\S+)", text).group(1)] = text
        at += 24
    return found


def test_no_sweep_uses_scratch(tmp_path):
    sweeps = {name: text for name, text in kernels(tmp_path).items() if "k_sweep" in name}
    # three dimensions: two modes and two directions alone and in batches, the barycentric rows
    assert len(sweeps) == 3 * (2 * 2 * 2 + 1)
    for name, text in sweeps.items():
        for key in ("private_segment_fixed_size", "vgpr_spill_count"):
            assert re.search(rf"\.{key}:\s+(\d+)", text).group(1) == "0", (name, key)
