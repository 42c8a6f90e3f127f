"""CPU tests of what the compiler gave the product's kernels, read from the metadata of the built libtutti.so (the code
object's own note record): no kernel uses scratch memory, and every kernel of a whole-GPU launch fits eight times into a
compute unit, which is what those launches' grids are sized for."""
import re
import struct
import subprocess
import sys

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


def _short_names(mangled):
    """Kernel names without namespace and arguments."""
    names = subprocess.run(["c++filt"], input="\n".join(mangled), capture_output=True, text=True, check=True).stdout
    return [re.sub(r"\((tutti::|unsigned).*", "", n).replace("void ", "").replace("tutti::", "")
            for n in names.split("\n")[:len(mangled)]]


@pytest.fixture(scope="module")
def kernels():
    with open(B.LIB_PATH, "rb") as f:
        found = _metadata(_code_object(f.read()))["amdhsa.kernels"]
    return dict(zip(_short_names([k[".name"] for k in found]), found))


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


# Stands in for the two HIP calls by which kernels become known and are asked about, so that the query runs without a GPU.
RECORDER = """
#include <cstdio>
#include <map>
static std::map<const void *, const char *> names;
extern "C" void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *,
                                      void *, int *) { names[host] = name; }
extern "C" int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *host, int, size_t) {
  std::puts(names.at(host));
  std::fflush(stdout);
  *n = 8;
  return 0;
}
"""
ASK = """
import ctypes, sys
ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
for which in sys.argv[3:]:
    assert lib.tutti_resident_wgs_per_cu(int(which)) == 8
"""


@pytest.mark.parametrize("which,kernel", [((2, 3), "k_move<"), ((4, 5), "k_layer_ring<"), ((0, 1, 6, 7), "k_layer<"),
                                          ((10,), "k_issue_io<")], ids=lambda x: x if isinstance(x, str) else "")
def test_residency_query_asks_about_every_kernel(kernels, tmp_path, which, kernel):
    """tutti_resident_wgs_per_cu is the least over all kernels that a whole-GPU call of that kind may run."""
    source, stub = tmp_path / "recorder.cpp", tmp_path / "recorder.so"
    source.write_text(RECORDER)
    subprocess.run(["g++", "-shared", "-fPIC", str(source), "-o", str(stub)], check=True)
    out = subprocess.run([sys.executable, "-c", ASK, str(stub), B.LIB_PATH, *map(str, which)], capture_output=True, text=True,
                         check=True).stdout
    there = {n for n, k in kernels.items() if n.startswith(kernel) and k[".max_flat_workgroup_size"] == 256}
    assert set(_short_names(out.split())) == there and len(there) >= 2
