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
extern "C" unsigned units_of(int ahead, unsigned block_bytes, unsigned blocks, unsigned budget, int ordered,
                             int short_rows) {
  return tutti::budget_units(ahead != 0, block_bytes, blocks, budget, ordered != 0, short_rows != 0);
}
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
        assert rules.pause_of(items, CHIP, n_req, file) <= 8


def test_more_requests_are_held_back_less(rules):
    for items in range(0, 3 * CHIP, 64):
        pauses = [rules.pause_of(items, CHIP, n, 0) for n in range(1, 65)]
        assert pauses == sorted(pauses, reverse=True)
    assert [rules.pause_of(CHIP, CHIP, n, 0) for n in (1, 2, 8, 64)] == [8, 7, 6, 5]
    assert [rules.pause_of(CHIP * 7 // 8, CHIP, n, 0) for n in (1, 2, 8, 64)] == [6, 5, 4, 3]
    assert [rules.pause_of(CHIP * 3 // 4, CHIP, n, 0) for n in (1, 2, 8, 64)] == [2, 2, 1, 0]


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


def test_head_major_rows_through_lds(rules):
    """Every row below a cache line on the whole GPU, none of a line or more anywhere, and under a budget the shortest rows
    only, on more than 16 compute units."""
    for row in range(16, 512, 16):
        assert rules.lds_of(row, 0) == (row < 128)
        for budget in (1, 8, 16):
            assert not rules.lds_of(row, budget)
        for budget in (17, 32, 64, 256):
            assert rules.lds_of(row, budget) == (row == 16)
