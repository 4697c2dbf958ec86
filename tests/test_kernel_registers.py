"""What the compiler made of the bfloat16 GEMM's kernels, from the metadata and the code in the built library: the main loops rest
on register budgets, and their loads on a register that the compiler does not know to be in use, which nothing else checks."""
import os
import re
import shutil
import struct
import subprocess

import msgpack
import pytest

from paper_2506_22175_amd import build

NT_AMDGPU_METADATA, SHT_NOTE = 32, 7


def _code_objects(data):
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length]:
                yield data[at + offset:at + offset + size]
            p += 24 + length
        at = data.find(magic, at + 24)


@pytest.fixture(scope="module")
def objects():
    if not os.path.exists(build.OUT):
        build.build()
    return list(_code_objects(open(build.OUT, "rb").read()))


@pytest.fixture(scope="module")
def kernels(objects):
    """name -> metadata"""
    found = {}
    for obj in objects:
        (table,) = struct.unpack_from("<Q", obj, 0x28)
        size, count = struct.unpack_from("<HH", obj, 0x3a)
        for s in range(count):
            if struct.unpack_from("<I", obj, table + s * size + 4)[0] != SHT_NOTE:
                continue
            (at,) = struct.unpack_from("<Q", obj, table + s * size + 0x18)
            name, desc, kind = struct.unpack_from("<III", obj, at)
            if kind == NT_AMDGPU_METADATA:
                start = at + 12 + (name + 3) // 4 * 4
                for k in msgpack.unpackb(obj[start:start + desc])["amdhsa.kernels"]:
                    found[k[".name"]] = k
    return found


def test_no_vector_register_is_spilled(kernels):
    gemms = [k for name, k in kernels.items() if "gemm_" in name]
    assert len(gemms) >= 38
    for k in gemms:
        assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, k[".name"]


# (layout NN/NT/TN, epilogue: store, GeLU, GeLU-backward, float store, float sums, scattered; rows, columns): vector
# registers, spilled scalars.  A spilled scalar is a lane write and a lane read in a tile's prologue, which a launch of a
# tile or two per CU does not cover.
SMALLER_TILES = {
    (0, 0, 64, 64): (104, 33), (0, 0, 64, 128): (124, 26), (0, 0, 128, 128): (142, 9), (0, 0, 256, 128): (272, 63),
    (0, 1, 64, 128): (128, 37), (0, 1, 128, 128): (144, 28), (0, 1, 256, 128): (272, 91),
    (0, 5, 64, 64): (104, 39), (0, 5, 64, 128): (132, 34), (0, 5, 128, 128): (143, 22), (0, 5, 256, 128): (276, 74),
    (1, 0, 64, 128): (172, 29), (1, 0, 128, 128): (148, 10), (1, 0, 256, 128): (304, 65),
    (1, 2, 64, 128): (172, 92), (1, 2, 128, 128): (181, 69), (1, 2, 256, 128): (320, 177),
    (2, 3, 128, 128): (139, 28), (2, 3, 256, 128): (280, 61), (2, 4, 128, 128): (139, 23), (2, 4, 256, 128): (248, 53),
}
# 256 x 256 weight gradients: the descriptors carry K, so that neither offsets nor lanes are formed again for every tile and range
LARGE_WEIGHT_GRADIENTS = {(2, 3, 256, 256): (468, 68), (2, 4, 256, 256): (400, 50)}


@pytest.mark.parametrize("bounds", [SMALLER_TILES, LARGE_WEIGHT_GRADIENTS], ids=["smaller_tiles", "large_weight_gradients"])
def test_tiles_keep_within_their_registers(kernels, bounds):
    """What the 256 x 256 tiles' loops need (offsets to carry along) must not end up in the smaller tiles."""
    seen = {}
    for name, k in kernels.items():
        m = re.search(r"gemm_bf16_kernelILi(\d)ELi(\d)ENS_7TileCfgILi(\d+)ELi(\d+)E", name)
        if m:
            seen[tuple(int(v) for v in m.groups())] = (k[".vgpr_count"], k[".sgpr_spill_count"])
    for kernel, (registers, spilled) in bounds.items():
        assert seen[kernel][0] <= registers and seen[kernel][1] <= spilled, (kernel, seen[kernel])


def _objdump():
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    for root in (os.path.dirname(os.path.dirname(os.path.realpath(hipcc))), "/opt/rocm"):
        tool = os.path.join(root, "llvm", "bin", "llvm-objdump")
        if os.path.exists(tool):
            return tool
    pytest.skip("no disassembler for gfx950")


def test_every_load_into_lds_has_the_address_that_was_set_for_it(objects, tmp_path):
    """m0 holds the LDS address of a buffer load into LDS.  The kernels set it in assembly, some loads one or more instructions
    later, and the compiler, for which m0 cannot be named as changed or read by such a statement, could write it in between."""
    loads = 0
    for i, obj in enumerate(objects):
        path = tmp_path / f"{i}.co"
        path.write_bytes(obj)
        text = subprocess.run([_objdump(), "-d", "--no-show-raw-insn", str(path)], capture_output=True, text=True, check=True).stdout
        for kernel in re.split(r"\n(?=[0-9a-f]{16} <)", text):
            if "gemm_bf16" not in kernel.split("\n", 1)[0]:
                continue
            code = [re.sub(r"\s*//.*", "", line).strip() for line in kernel.splitlines()[1:]]
            code = [line for line in code if line]
            set_at = None                              # where m0 was written for a load to come
            for at, line in enumerate(code):
                if re.match(r"buffer_load_dwordx4 .*\blds$", line):
                    assert set_at is not None and at - set_at >= 2, (line, code[max(0, at - 4):at])
                    loads, set_at = loads + 1, None
                elif re.search(r"\bm0\b", line):
                    # either statement that sets it, and only once for a load
                    assert re.match(r"s_add_u32 m0, (m0, 0x400|s\d+, )", line) or \
                        (re.match(r"s_mov_b32 m0, ", line) and code[at + 1] == "s_nop 0" and code[at + 2].endswith(" lds")), line
                    assert set_at is None, code[set_at:at + 1]
                    set_at = at
            assert set_at is None
    assert loads > 1000
