"""CPU tests of what the compiler gave the product's kernels, read from the metadata of the built libtutti.so (the code
object's own note record): no kernel uses scratch memory, and every kernel of a whole-GPU launch fits eight times into a
compute unit, which is what those launches' grids are sized for."""
import re
import struct
import subprocess

import msgpack
import pytest

from paper_2605_03375_amd import binding as B

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_object(blob):
    """The gfx950 code object inside the library's offload bundle."""
    at = blob.index(BUNDLE)
    n, = struct.unpack_from("<Q", blob, at + len(BUNDLE))
    pos = at + len(BUNDLE) + 8
    for _ in range(n):
        offset, size, name_len = struct.unpack_from("<QQQ", blob, pos)
        name = blob[pos + 24:pos + 24 + name_len].decode()
        pos += 24 + name_len
        if "gfx950" in name:
            return blob[at + offset:at + offset + size]
    raise AssertionError("no gfx950 code object in the library")


def _metadata(elf):
    """The note record that describes the kernels (AMDGPU metadata, a msgpack map)."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    entsize, count = struct.unpack_from("<HH", elf, 0x3a)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + i * entsize + 4)
        offset, size = struct.unpack_from("<QQ", elf, shoff + i * entsize + 24)
        end = offset + size
        while kind == 7 and offset < end:  # SHT_NOTE
            name_len, desc_len, note = struct.unpack_from("<III", elf, offset)
            desc = offset + 12 + (name_len + 3) // 4 * 4
            if note == 32:                 # NT_AMDGPU_METADATA
                return msgpack.unpackb(elf[desc:desc + desc_len], raw=False)
            offset = desc + (desc_len + 3) // 4 * 4
    raise AssertionError("no kernel metadata")


@pytest.fixture(scope="module")
def kernels():
    with open(B.LIB_PATH, "rb") as f:
        found = _metadata(_code_object(f.read()))["amdhsa.kernels"]
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), capture_output=True, text=True,
                           check=True).stdout.split("\n")
    return {re.sub(r"\((tutti::|unsigned).*", "", n).replace("void ", "").replace("tutti::", ""): k
            for n, k in zip(names, found)}


def test_no_kernel_uses_scratch(kernels):
    """Scratch is memory: a kernel of 8192 wavefronts that spills 36 bytes a lane moves 19 MB on the side."""
    assert len(kernels) > 20 and any(n.startswith("k_layer<") for n in kernels)
    bad = {n: (k[".private_segment_fixed_size"], k[".vgpr_spill_count"]) for n, k in kernels.items()
           if k[".private_segment_fixed_size"] != 0 or k[".vgpr_spill_count"] != 0}
    assert not bad, f"scratch bytes a lane, spilled vector registers: {bad}"


def test_whole_gpu_kernels_fit_eight_times(kernels):
    """Eight workgroups of 256 threads a compute unit are eight wavefronts a SIMD, which have 64 vector registers each:
    every copy kernel of that workgroup size, whatever the number of requests, the blocks or the order it is for."""
    whole = {n: k for n, k in kernels.items() if k[".max_flat_workgroup_size"] == 256 and
             re.match(r"k_layer<|k_layer_ring<|k_move<|k_issue_io<|k_layer_lds<., [124],|k_move_lds<., [124],", n)}
    assert len({n.split("<")[0] for n in whole}) == 6 and len(whole) > 40
    large = {n: k[".vgpr_count"] for n, k in whole.items() if k[".vgpr_count"] > 64}
    assert not large, large
