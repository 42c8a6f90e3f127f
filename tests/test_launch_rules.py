"""CPU tests of the rules by which a call's kernel and launch shape are chosen (csrc/launch_rules.h)."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "launch_rules.h"
extern "C" unsigned pause_of(unsigned items, unsigned chip, unsigned n_req, int file) {
  return tutti::hold_back_pause(items, chip, n_req, file != 0);
}
extern "C" int lds_of(unsigned row, unsigned budget) { return tutti::hnd_through_lds(row, budget); }
extern "C" int tiles_of(unsigned row, unsigned block_bytes, unsigned heads, unsigned budget, int unpack, int half_empty) {
  return tutti::as_line_tiles(row, block_bytes, heads, budget, unpack != 0, half_empty != 0);
}
extern "C" unsigned tile_shift_of(unsigned row_shift, unsigned head_shift, unsigned token_shift) {
  return tutti::line_tile_shift(row_shift, head_shift, token_shift);
}
extern "C" int apart_of(unsigned copy_wgs, unsigned cus, unsigned n_req) {
  return tutti::entries_apart(copy_wgs, cus, n_req);
}
extern "C" unsigned units_of(int ahead, unsigned block_bytes, unsigned blocks, unsigned budget, int ordered,
                             int short_rows) {
  return tutti::budget_units(ahead != 0, block_bytes, blocks, budget, ordered != 0, short_rows != 0);
}
extern "C" int at_once_of(unsigned long long items, unsigned chip, unsigned n_req, unsigned table_len) {
  return tutti::pack_at_once(items, chip, n_req, table_len);
}
extern "C" unsigned cut_of(unsigned block_bytes) { return tutti::cut_slice(block_bytes); }
extern "C" int cuts_of(int unpack, unsigned n_req, unsigned block, unsigned slice, unsigned long long items, unsigned chip) {
  return tutti::cuts_blocks(unpack != 0, n_req, block, slice, items, chip);
}
extern "C" unsigned grid_of(unsigned cus, unsigned wgs_per_cu) { return tutti::full_grid(cus, wgs_per_cu); }
extern "C" int one_slice_of(unsigned long long items, unsigned long long chip) { return tutti::one_slice_saves(items, chip); }
extern "C" int pieces_of(int whole_gpu, unsigned units) { return tutti::pieces_shape(whole_gpu != 0, units); }
"""
CHIP = 8192  # wavefronts of a whole-GPU launch on 256 compute units


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, lib = d / "rules.cpp", d / "rules.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC",
                    f"-I{ROOT}/paper_2605_03375_amd/csrc", str(src), "-o", str(lib)], check=True)
    return ctypes.CDLL(str(lib))


@pytest.mark.parametrize("file", [0, 1])
@pytest.mark.parametrize("n_req", [1, 2, 8, 64])
def test_stores_are_held_back_by_the_items_there_are(rules, n_req, file):
    """Never for a job that leaves a third of the chip free (whatever its table could hold) or that gives a wavefront
    more than two items; never without a chip size (under a budget)."""
    for items in (0, 1, 64, 1024, CHIP // 2, CHIP * 21 // 32, 2 * CHIP + 1, 4 * CHIP, 0x7fffffff, 0xffffffff):
        assert rules.pause_of(items, CHIP, n_req, file) == 0
    for items in (0, 1, CHIP, 0xffffffff):
        assert rules.pause_of(items, 0, n_req, file) == 0
    for items in range(CHIP // 2, 2 * CHIP + 64, 16):
        assert rules.pause_of(items, CHIP, n_req, file) <= 9


def test_more_requests_are_held_back_less(rules):
    for items in range(0, 3 * CHIP, 64):
        pauses = [rules.pause_of(items, CHIP, n, 0) for n in range(1, 65)]
        assert pauses == sorted(pauses, reverse=True)
    # behind the step that the time falls off at each size
    assert [rules.pause_of(CHIP, CHIP, n, 0) for n in (1, 2, 8, 32, 33, 64)] == [9, 9, 9, 9, 8, 8]
    assert [rules.pause_of(CHIP * 29 // 32, CHIP, n, 0) for n in (1, 2, 8, 64)] == [9, 9, 9, 8]
    assert [rules.pause_of(CHIP * 7 // 8, CHIP, n, 0) for n in (1, 2, 8, 64)] == [6, 6, 6, 6]
    assert [rules.pause_of(CHIP * 3 // 4, CHIP, n, 0) for n in (1, 2, 8, 64)] == [2, 2, 2, 2]
    assert [rules.pause_of(CHIP * 5 // 4, CHIP, n, 0) for n in (1, 2, 8, 64)] == [8, 8, 8, 8]


@pytest.mark.parametrize("ahead", [0, 1])
@pytest.mark.parametrize("budget", [1, 8, 16, 32, 64, 256])
def test_slices_under_a_budget(rules, ahead, budget):
    """A visiting order never cuts a block of whole 8 KiB slices into anything else, and gets 8 KiB slices otherwise;
    without one a slice fills the blocks, or the block goes as pieces 16 at a time."""
    for kib4 in range(1, 65):
        for extra in (0, 16, 512, 1024):
            block = 4096 * kib4 + extra
            for blocks in (0, 1, 64, 512, 513, 4096, 1 << 20, 0xffffffff):
                u = rules.units_of(ahead, block, blocks, budget, 1, 0)
                assert u in (8, 16) and (u == 8 or block % 16384 == 0)
                v = rules.units_of(ahead, block, blocks, budget, 0, 0)
                assert v in (8, 16) and (v == 16 or block % 8192 == 0)
                if ahead and block % 16384 == 8192:
                    assert v == 8
    assert [rules.units_of(1, 32768, 34, b, 0, 0) for b in (8, 16, 32, 64)] == [16, 16, 8, 8]
    for blocks in (1, 64, 256, 512):
        assert rules.units_of(1, 32768, blocks, 32, 0, 0) == (16 if blocks > 256 else 8)
        assert rules.units_of(ahead, 32768, blocks, budget, 0, 1) == rules.units_of(ahead, 16384, blocks, budget, 1, 1) == 16


@pytest.mark.parametrize("ahead,short_rows", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("budget", [1, 16, 32, 256])
def test_ragged_blocks_have_a_kernel(rules, ahead, short_rows, budget):
    """Where the slices that the rule asks for do not fill the blocks, the shape is one that moves pieces."""
    ragged = 0
    for block in [16 * k for k in range(1, 1100)] + [1024 * k for k in range(18, 256)]:
        for blocks in (1, 64, 513, 4096, 1 << 20):
            units = rules.units_of(ahead, block, blocks, budget, 0, short_rows)
            if block % (units * 1024) != 0:
                ragged += 1
                assert rules.pieces_of(0, units)
        assert rules.pieces_of(1, 4)
    assert ragged > 1000 and not rules.pieces_of(0, 8)


def test_head_major_rows_through_lds(rules):
    """Every row below a cache line on the whole GPU, none of a line or more anywhere, and under a budget the shortest rows
    only, on more than 16 compute units."""
    for row in range(16, 512, 16):
        assert rules.lds_of(row, 0) == (row < 128)
        for budget in (1, 8, 16):
            assert not rules.lds_of(row, budget)
        for budget in (17, 32, 64, 256):
            assert rules.lds_of(row, budget) == (row == 16)


def test_line_tiles_cover_the_block(rules):
    """Every shape that the rule takes: the tiles are whole, deal out every 16 bytes of the block once on both sides, and
    touch whole lines on both wherever tokens and heads are enough for it."""
    taken = 0
    for rs in range(4, 10):
        for hs in range(0, 8):
            for ts in range(0, 9):
                if not rules.tiles_of(1 << rs, 1 << (rs + hs + ts), 1 << hs, 0, 1, 1):
                    assert rs + hs + ts < 12
                    continue
                taken += 1
                tg = rules.tile_shift_of(rs, hs, ts)
                hg = 10 - rs - tg
                assert 0 <= tg <= ts and 0 <= hg <= hs
                assert tg + rs >= 7 or tg == ts
                assert hg + rs >= 7 or hg == hs
                if ts + hs + rs > 14:
                    continue
                pool, obj = set(), set()
                for q in range(1 << (rs + hs + ts - 10)):
                    heads, tokens = q & ((1 << (hs - hg)) - 1), q >> (hs - hg)
                    for lane in range(64):
                        w, t = lane & ((1 << (rs - 4)) - 1), lane >> (rs - 4) & ((1 << tg) - 1)
                        i = lane >> (rs - 4 + tg)
                        i, t = (heads << hg) + i, (tokens << tg) + t
                        pool.add((((i << ts) + t) << rs) + 16 * w)
                        obj.add((((t << hs) + i) << rs) + 16 * w)
                assert pool == obj == set(range(0, 1 << (rs + hs + ts), 16))
    assert taken > 80
    assert not rules.tiles_of(128, 32768, 16, 0, 0, 0) and not rules.tiles_of(64, 16384, 8, 32, 1, 0)
    assert not rules.tiles_of(1024, 32768, 16, 0, 0, 1) and not rules.tiles_of(256, 32768, 16, 8, 0, 1)
    assert rules.tiles_of(64, 16384, 8, 32, 0, 0) and rules.tiles_of(64, 16384, 16, 32, 1, 0)


def test_entries_apart_from_small_launches_only(rules):
    for cus in (1, 8, 256):
        for n_req, last in ((1, 2 * cus), (2, 5 * cus // 2), (64, 5 * cus // 2)):
            assert rules.apart_of(1, cus, n_req) and rules.apart_of(last, cus, n_req)
            assert not rules.apart_of(last + 1, cus, n_req) and not rules.apart_of(8 * cus, cus, n_req)


def test_long_tables_are_counted_first(rules):
    """Up to 64 requests beyond a quarter of the chip; of more, tables of more than 8 blocks a request."""
    rules.at_once_of.argtypes = [ctypes.c_ulonglong] + [ctypes.c_uint] * 3
    for n_req, longest in ((2, 0), (64, 0), (65, 520), (512, 4096), (1024, 8192), (1025, 0), (2048, 0)):
        for table in (1, 8, 520, 521, 4096, 4097, 8192, 8193, 0xffffffff):
            assert rules.at_once_of(CHIP // 4, CHIP, n_req, table)
            assert rules.at_once_of(CHIP // 4 + 1, CHIP, n_req, table) == (table <= longest)
            assert rules.at_once_of(1 << 33, CHIP, n_req, table) == (table <= longest)


def test_cut_slices_fill_the_block(rules):
    """Whole lines, at most the 4 KiB of a wavefront's accesses, as few as can be and none left over; none for blocks without
    such slices."""
    cut = 0
    for block in [*range(16, 1 << 16, 16), *range(1 << 16, 1 << 20, 128), 0xfffffff0, 0xffffff80]:
        b = rules.cut_of(block)
        if b:
            cut += 1
            assert block % b == 0 and b % 128 == 0 and b <= 4096
            assert b == block or b > 1024
            assert not [n for n in range(-(-block // 4096), block // b) if block % (128 * n) == 0]
        else:
            assert block % 128 or not 1024 <= block <= 512 << 10 or \
                not [n for n in range(-(-block // 4096), 2 * -(-block // 4096)) if block % (128 * n) == 0]
    assert cut > 1000
    assert [rules.cut_of(b) for b in (1024, 2560, 6400, 12800, 15360, 30720)] == [1024, 2560, 3200, 3200, 3840, 3840]


def test_blocks_are_cut_up_to_a_slice_a_wavefront(rules):
    rules.cuts_of.argtypes = [ctypes.c_int] + [ctypes.c_uint] * 3 + [ctypes.c_ulonglong, ctypes.c_uint]
    for unpack, n_req, block, most in ((0, 1, 12800, 2 * CHIP), (0, 2, 12800, CHIP), (0, 300, 2176, CHIP), (1, 1, 6400, CHIP),
                                       (1, 65, 12800, CHIP), (1, 65, 15360, CHIP // 2), (0, 1, 2048, CHIP // 2),
                                       (0, 65, 1024, CHIP // 2), (1, 1, 1024, CHIP // 4), (1, 2, 2048, CHIP // 4)):
        slice_ = rules.cut_of(block)
        assert rules.cuts_of(unpack, n_req, block, slice_, 0, CHIP) and rules.cuts_of(unpack, n_req, block, slice_, most, CHIP)
        assert not rules.cuts_of(unpack, n_req, block, slice_, most + 1, CHIP)
        assert not rules.cuts_of(unpack, n_req, block, slice_, 1 << 33, CHIP)


@pytest.mark.parametrize("cus", [1, 64, 256, 304])
def test_saves_of_one_slice_a_wavefront_have_the_wavefronts(rules, cus):
    """With every workgroup count that the knob takes: the rule admits no more slices than the launched grid has wavefronts, and
    the grid is one that the arguments' fields hold."""
    rules.one_slice_of.argtypes = [ctypes.c_ulonglong] * 2
    for per_cu in [*range(1, 40), 64, 256, 1024]:
        most = rules.grid_of(cus, per_cu)
        assert most == min(cus * per_cu, 4088)
        assert rules.one_slice_of(3 * most, 4 * most)
        for items in range(3 * most - 8, 4 * cus * per_cu + 8, 61):
            grid = min(-(-items // 4), most)
            if rules.one_slice_of(items, 4 * most):
                assert items <= 4 * grid, (per_cu, items)
