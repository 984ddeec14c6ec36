"""What no result shows of the built kernels, read from their code objects (no
GPU): registers that the launch rules count on (a few too many halve the
work-groups a compute unit holds), and waits in the march of the planes."""
import os
import re
import struct
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_objects(wave_mod, tmp_path_factory):
    """The library's gfx950 code objects, as files."""
    d = tmp_path_factory.mktemp("co")
    fat = d / "fat"
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", wave_mod.LIB_PATH, str(d / "x")],
                   check=True)
    data = fat.read_bytes()
    out = []
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        (n,), at = struct.unpack_from("<Q", data, m.end()), m.end() + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" in target and size:
                out.append(d / f"elf{len(out)}")
                out[-1].write_bytes(data[m.start() + off:m.start() + off + size])
    return out


def tool(name, *args):
    return subprocess.run([f"{LLVM}/{name}", *map(str, args)], check=True, capture_output=True, text=True).stdout


@pytest.fixture(scope="module")
def kernels(code_objects):
    """{mangled kernel name: (VGPRs, scratch bytes, code object)}"""
    out = {}
    for elf in code_objects:
        for k in tool("llvm-readelf", "--notes", elf).split("- .agpr_count")[1:]:
            vgprs, scratch = (int(re.search(rf"\.{f}:\s+(\d+)", k)[1])
                              for f in ("vgpr_count", "private_segment_fixed_size"))
            out[re.search(r"\.name:\s+(\S+)", k)[1]] = vgprs, scratch, elf
    return out


def named(kernels, kernel, args):
    prefix = f"_ZN5wavek{len(kernel)}{kernel}I" + "".join(f"Li{a}E" for a in args) + "E"
    name, = [n for n in kernels if n.startswith(prefix)]
    return name, kernels[name]


needs_tools = pytest.mark.skipif(not os.path.exists(f"{LLVM}/llvm-objcopy"), reason="no LLVM tools")


# 128 registers: four waves a SIMD, two work-groups of 512 threads a CU
@needs_tools
@pytest.mark.parametrize("tile", [(16, 16, 1), (16, 32, 1), (32, 16, 1)])
@pytest.mark.parametrize("kernel,args", [("step_batch", (0,)), ("step_tiled", (0,)), ("step_tiled_cached", ())])
def test_fp32_one_row_tiles_leave_room_for_four_waves(kernels, kernel, args, tile):
    _, (vgprs, scratch, _) = named(kernels, kernel, args + tile)
    assert vgprs <= 128 and scratch == 0


# the march issues the next plane's loads, then writes this one's halo to LDS: a
# wait for every load there is one for the loads just issued
@needs_tools
@pytest.mark.parametrize("kernel,args", [
    (k, (kind, *tile)) for k in ("step_batch", "step_batch_run") for kind in (0, 1, 2)
    for tile in ((64, 8, 1), (32, 16, 1), (16, 16, 1), (32, 8, 2))] + [("step_tiled", (0, 64, 8, 1))])
def test_march_does_not_wait_for_the_next_plane(kernels, kernel, args):
    name, (_, _, elf) = named(kernels, kernel, args)
    code = [line.split("//")[0].strip() for line in
            tool("llvm-objdump", "-d", "--mcpu=gfx950", f"--disassemble-symbols={name}", elf).splitlines()]
    assert sum(c.startswith("buffer_load") for c in code) > 50
    drained = [i for i, (a, b) in enumerate(zip(code, code[1:]))
               if a.startswith("s_waitcnt") and "vmcnt(0)" in a and b.startswith("ds_write")]
    assert not drained
