"""CPU test of the rules by which saves, and restores of one request, hold their first stores back (csrc/launch_rules.h)."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "launch_rules.h"
extern "C" unsigned pause_of(int which, unsigned items, unsigned chip, unsigned n_req) {
  return which == 0 ? tutti::one_restore_pause(items, chip)
         : which == 1 ? tutti::one_save_pause(items, chip) : tutti::few_save_pause(items, chip, n_req);
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("pauses")
    src, lib = d / "pauses.cpp", d / "pauses.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC",
                    f"-I{ROOT}/paper_2605_03375_amd/csrc", str(src), "-o", str(lib)], check=True)
    return ctypes.CDLL(str(lib))


@pytest.mark.parametrize("which, first, last", [(0, 7, 32), (1, 9, 22.5), (2, 9, 32)])
@pytest.mark.parametrize("chip", [8192, 1024])
def test_pause_grows_with_the_items_and_has_an_end(rules, which, first, last, chip):
    """Between `first` and `last` 32nds of the chip's wavefronts only; no step back; never without a chip size."""
    for n_req in (1, 32, 33, 64):
        before = 0
        for items in range(0, chip + 1, chip // 1024):
            p = rules.pause_of(which, items, chip, n_req)
            assert (p > 0) == (first * chip <= 32 * items <= last * chip), items
            assert p >= before or p == 0
            assert p <= 14
            before = p
        for items in (chip + 1, 1 << 27, (1 << 27) + chip // 2, 0x7fffffff, 0xffffffff):  # 32 * items passes 2^32
            assert rules.pause_of(which, items, chip, n_req) == 0
        for items in (0, 1, chip, 0xffffffff):
            assert rules.pause_of(which, items, 0, n_req) == 0


LINES = """
#include "launch_rules.h"
extern "C" unsigned lines_pause_of(int few, unsigned items, unsigned chip, int lines) {
  return few ? tutti::few_save_pause(items, chip, 9, lines != 0) : tutti::one_save_pause(items, chip, lines != 0);
}
"""


@pytest.mark.parametrize("few, none", [(0, (20.5, 22.5)), (1, (12, 16))])
def test_line_tiles_are_not_held_back_where_that_costs(tmp_path, few, none):
    """Line tiles: no pause in the part of the range (in 32nds of the chip) where other saves have one, the same elsewhere."""
    src, lib = tmp_path / "lines.cpp", tmp_path / "lines.so"
    src.write_text(LINES)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC",
                    f"-I{ROOT}/paper_2605_03375_amd/csrc", str(src), "-o", str(lib)], check=True)
    pause = ctypes.CDLL(str(lib)).lines_pause_of
    for chip in (8192, 1024):
        for items in range(chip + 1):
            i = 32 * items
            inside = none[0] * chip < i <= none[1] * chip or (few and i == none[0] * chip)
            assert pause(few, items, chip, 1) == (0 if inside else pause(few, items, chip, 0)), items
