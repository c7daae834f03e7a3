"""Lists of limited rows (csrc/row_lists.hpp), built for the host: every
block's rows have room whatever the marked rows are, blocks of a mesh line
spread over the lists, and the waves' parts are equal."""
import ctypes as C
import subprocess

import numpy as np
import pytest

from paper_2106_02159_amd import build as B

PROGRAM = """
#define __host__
#define __device__
#include "row_lists.hpp"
using namespace ns;
extern "C" void plan(uint32_t blocks, uint32_t *out, uint32_t *list) {
  const RowLists rl(blocks);
  out[0] = rl.lists;
  out[1] = rl.room;
  for (uint32_t b = 0; b < blocks; ++b) list[b] = rl.list_of(b);
}
extern "C" void rows_of(uint32_t lists, const uint32_t *len, uint32_t groups, int *group) {
  uint32_t longest = 0;
  for (uint32_t l = 0; l < lists; ++l) longest = len[l] > longest ? len[l] : longest;
  const uint32_t each = part_rows(longest, lists, groups);
  for (uint32_t b = 0; b < groups; ++b)
    for (uint32_t p = b; p / lists * each < longest; p += groups)
      for (uint32_t t = p / lists * each; t < (p / lists + 1) * each && t < len[p % lists]; ++t)
        ++group[b];
}
"""


@pytest.fixture(scope="module")
def lists(tmp_path_factory):
    d = tmp_path_factory.mktemp("lists")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text("#pragma once\n")
    (d / "lists.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I", str(d), "-I", B.CSRC,
                    str(d / "lists.cpp"), "-o", str(d / "lists.so")], check=True)
    return C.CDLL(str(d / "lists.so"))


def ptr(a):
    return a.ctypes.data_as(C.c_void_p)


def plan(lib, blocks):
    out, of = np.zeros(2, np.uint32), np.zeros(blocks, np.uint32)
    lib.plan(blocks, ptr(out), ptr(of))
    return int(out[0]), int(out[1]), of


def test_room(lists):
    """All rows marked: no list holds more than its room, and the lists fit the
    work-list array of 9 words per row in slices of 64."""
    for blocks in list(range(1, 300)) + [1023, 4096, 65537, 66400]:
        n, room, of = plan(lists, blocks)
        assert n <= 64 and of.max() < n
        assert np.bincount(of, minlength=n).max() * 256 <= room
        fewest = 64 * (4 * (blocks - 1) + 1)  # rows of that many blocks, at least
        assert n * room <= 9 * fewest
        assert 64 * 8 <= 9 * fewest  # the lists' counters


@pytest.mark.parametrize("nx,ny", [(4096, 4096), (4096, 4150), (4096, 4022), (4096, 4086),
                                   (2368, 2432), (1024, 1061), (3000, 301), (257, 4096),
                                   (97, 83), (60, 60), (5, 7)])
def test_fronts(lists, nx, ny):
    """Fronts along x and along y, and all rows: the appends of a list's counter
    and the rows of a workgroup stay near their means."""
    blocks = -(-nx * ny // 256)
    n, room, of = plan(lists, blocks)
    rows = np.arange(nx * ny)
    groups = min(512, -(-nx * ny // 64))
    marks = [np.ones(nx * ny, bool)]
    for at in (0.3, 0.5, 0.77):
        marks += [np.abs(rows % nx - at * nx) <= 4, np.abs(rows // nx - at * ny) <= 4]
    for marked in marks:
        hit = np.unique(rows[marked] // 256)
        per = np.bincount(of[hit], minlength=n)
        # (a hash's spread: the mean and some standard deviations of it)
        assert per.max() <= len(hit) / n + 5.0 * np.sqrt(len(hit) / n) + 2
        length = np.bincount(of[rows[marked] // 256], minlength=n).astype(np.uint32)
        count = np.zeros(groups, np.int32)
        lists.rows_of(n, ptr(length), groups, ptr(count))
        assert count.sum() == marked.sum()
        assert count.max() <= 2 * marked.sum() / groups + 64
