"""Registers of the built kernels that the launch rules count on, read from the
code object's own metadata (no GPU): a few registers too many halve the
work-groups a compute unit holds, which no result shows."""
import os
import re
import struct
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(wave_mod, tmp_path_factory):
    """{mangled kernel name: (VGPRs, scratch bytes)}"""
    d = tmp_path_factory.mktemp("co")
    fat = d / "fat"
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", wave_mod.LIB_PATH, str(d / "x")],
                   check=True)
    data = fat.read_bytes()
    out = {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        (n,), at = struct.unpack_from("<Q", data, m.end()), m.end() + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" not in target or not size:
                continue
            elf = d / "elf"
            elf.write_bytes(data[m.start() + off:m.start() + off + size])
            notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(elf)], check=True, capture_output=True,
                                   text=True).stdout
            for k in notes.split("- .agpr_count")[1:]:
                out[re.search(r"\.name:\s+(\S+)", k)[1]] = tuple(
                    int(re.search(rf"\.{f}:\s+(\d+)", k)[1]) for f in ("vgpr_count", "private_segment_fixed_size"))
    return out


needs_tools = pytest.mark.skipif(not os.path.exists(f"{LLVM}/llvm-objcopy"), reason="no LLVM tools")


# 128 registers: four waves a SIMD, two work-groups of 512 threads a CU
@needs_tools
@pytest.mark.parametrize("tile", [(16, 16, 1), (16, 32, 1), (32, 16, 1)])
@pytest.mark.parametrize("kernel,args", [("step_batch", (0,)), ("step_tiled", (0,)), ("step_tiled_cached", ())])
def test_fp32_one_row_tiles_leave_room_for_four_waves(kernels, kernel, args, tile):
    prefix = f"_ZN5wavek{len(kernel)}{kernel}I" + "".join(f"Li{a}E" for a in args + tile) + "E"
    (vgprs, scratch), = [v for name, v in kernels.items() if name.startswith(prefix)]
    assert vgprs <= 128 and scratch == 0
