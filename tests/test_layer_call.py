"""CPU test of the bit fields in which a fused launch's arguments reach the kernel (csrc/layer_call.h)."""
import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
U64 = ("k_base", "v_base", "stage", "sqe", "table", "n_blocks", "extents", "totals", "file_id", "status", "block_stride",
       "stage_cap", "stage_addr")
U32 = ("num_blocks", "table_len", "block_bytes", "chunk_bytes", "sqe_cap", "sgl_id", "layer", "n_req", "align", "sqe_wgs",
       "copy_wgs", "copy_first", "chip_waves", "dense", "xcd_contiguous", "size_a", "size_b", "left_out")


class Fields(ctypes.Structure):
    _fields_ = [(n, ctypes.c_uint64) for n in U64] + [(n, ctypes.c_uint32) for n in U32]


SOURCE = """
#include "layer_call.h"
extern "C" unsigned long size_of_fields() { return sizeof(tutti::LayerFields); }
extern "C" void there_and_back(const tutti::LayerFields *in, tutti::LayerFields *out) { *out = tutti::unpack(tutti::pack(*in)); }
extern "C" void sizes(unsigned tokens, unsigned heads, unsigned row, int powers, unsigned *out) {
  tutti::LayerFields f{};
  f.block_bytes = tokens * heads * row;
  f.align = 16;
  tutti::put_sizes(f, tutti::BlockSizes{tokens, heads, row});
  const tutti::BlockSizes b = tutti::get_sizes(tutti::unpack(tutti::pack(f)), powers != 0);
  out[0] = b.tokens, out[1] = b.heads, out[2] = b.row_bytes;
}
extern "C" void blocks(unsigned long stride, unsigned num_blocks, tutti::LayerFields *out) {
  tutti::LayerFields f{};
  f.align = 16;
  const tutti::PoolBlocks b = tutti::blocks_in_memory(stride, num_blocks);
  f.block_stride = b.stride, f.num_blocks = b.n;
  *out = tutti::unpack(tutti::pack(f));
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("call")
    src, out = d / "call.cpp", d / "call.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC",
                    f"-I{ROOT}/paper_2605_03375_amd/csrc", str(src), "-o", str(out)], check=True)
    return ctypes.CDLL(str(out))


# name: (largest value, step): every other field takes all values of its type
LIMITS = {n: ((1 << 47) - 16, 16) for n in ("k_base", "v_base", "stage", "sqe", "stage_cap")}
LIMITS |= {n: ((1 << 47) - 1, 1) for n in ("table", "n_blocks", "extents", "totals", "file_id", "status")}
LIMITS |= dict(block_stride=((1 << 47) - 16, 16), stage_addr=((1 << 64) - 16, 16), block_bytes=((1 << 32) - 16, 16),
               chunk_bytes=((1 << 32) - 16, 16), table_len=((1 << 31) - 1, 1), layer=(65535, 1), n_req=(2048, 1),
               sqe_wgs=(4088, 1), copy_wgs=(4088, 1), copy_first=(4095, 1), chip_waves=(127 * 128, 128), dense=(1, 1), xcd_contiguous=(1, 1),
               left_out=(2, 1), size_a=(1 << 14, 1), size_b=(1 << 14, 1))


def _value(rng, name, end):
    if name == "align":
        return 16 << (rng.randrange(28) if end is None else 27 * end)
    top, step = LIMITS.get(name, (0xffffffff, 1))
    low = 1 if name in ("sqe_wgs", "size_a", "size_b") else 0
    if end is not None:
        return top if end else low
    return rng.randint(low, top // step) * step


@pytest.mark.parametrize("seed", range(200))
def test_every_field_comes_back(lib, seed):
    """Random fields, and each field at either end of its range with the others at the opposite end."""
    assert lib.size_of_fields() == ctypes.sizeof(Fields)
    rng = random.Random(seed)
    special = (U64 + U32)[seed] if seed < len(U64 + U32) else None
    for flip in (0, 1):
        f = Fields()
        for n in U64 + U32:
            end = None if special is None else flip ^ (n == special)
            setattr(f, n, _value(rng, n, end))
        out = Fields()
        lib.there_and_back(ctypes.byref(f), ctypes.byref(out))
        for n in U64 + U32:
            assert getattr(out, n) == getattr(f, n), n


def test_what_the_fields_cannot_hold(lib):
    """Blocks that lie one below the other; staging without an end; a capacity that is no multiple of 16; more wavefronts."""
    f, out = Fields(align=4096, sqe_wgs=1, size_a=1, size_b=1), Fields()
    for stride in (-32768, -(1 << 47), (1 << 47) - 16):
        f.block_stride = stride & (1 << 64) - 1
        lib.there_and_back(ctypes.byref(f), ctypes.byref(out))
        assert out.block_stride == f.block_stride
    for cap, held in ((1 << 47, (1 << 47) - 16), ((1 << 64) - 1, (1 << 47) - 16), (4095, 4080), (15, 0)):
        f.stage_cap = cap
        lib.there_and_back(ctypes.byref(f), ctypes.byref(out))
        assert out.stage_cap == held
    f.chip_waves = 1 << 20
    lib.there_and_back(ctypes.byref(f), ctypes.byref(out))
    assert out.chip_waves == 127 * 128


@pytest.mark.parametrize("stride, held", [(32768, True), ((1 << 47) - 16, True), ((1 << 64) - 32768, True),
                                          ((1 << 64) - (1 << 47), True), (1 << 47, False), ((1 << 48) + 4096, False),
                                          (1 << 60, False), (1 << 63, False), ((1 << 64) - (1 << 47) - 16, False)])
@pytest.mark.parametrize("num_blocks", [1, 2, 0xffffffff])
def test_blocks_are_where_the_stride_says_or_nowhere(lib, stride, held, num_blocks):
    """No id below the count that the kernel gets lies elsewhere than id * stride says."""
    out = Fields()
    lib.blocks(ctypes.c_ulong(stride), num_blocks, ctypes.byref(out))
    assert out.num_blocks == (num_blocks if held else 1)
    for b in (0, 1, out.num_blocks - 1):
        if b < out.num_blocks:
            assert (b * out.block_stride) % (1 << 64) == (b * stride) % (1 << 64)


# (tokens, heads, bytes of a row): the largest size that a field holds, one more beside it, and the longest ones
SHAPES = [(16, 8, 256), (16, 5, 160), (1, 1, 16), (16, 64, 16), (1 << 14, (1 << 14) - 1, 16), ((1 << 14) - 1, 1 << 14, 16),
          (1 << 14, 1 << 13, 16), ((1 << 14) + 1, 1 << 13, 16), (1 << 12, 3, 16 << 14), ((1 << 28) - 1, 1, 16),
          (1, (1 << 28) - 1, 16), (1, 1, (1 << 32) - 16), (3, 5, 16 * 65537), (1, 2, 16 << 26), (1 << 20, 2, 32), (2, 1 << 20, 32),
          (127, 129, 16 * 16383)]


@pytest.mark.parametrize("tokens, heads, row", SHAPES)
def test_block_sizes_come_back(lib, tokens, heads, row):
    assert tokens * heads * row < 1 << 32
    powers = all(x & (x - 1) == 0 for x in (tokens, heads, row))
    for p in (0, 1) if powers else (0,):
        out = (ctypes.c_uint32 * 3)()
        lib.sizes(tokens, heads, row, p, out)
        assert tuple(out) == (tokens, heads, row)
