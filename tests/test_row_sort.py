"""Which rows the build sorts by bitmap, and the launch sizes that follow, over
the whole accepted range: the host rules of csrc/row_sort.h, compiled alone."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MOST_THREADS = 1 << 32  # of a launch, in one dimension
MOST_ENTRIES = 1 << 31  # 2 per input pair, at most 2^30 pairs
MOST_NODES = (1 << 31) - 2

SHIM = """
#include "row_sort.h"
using namespace tricc;
extern "C" {
int32_t ranges(int64_t n) { return row_ranges(n); }
int32_t bitmap_min(int64_t n) { return row_bitmap_min(n); }
int first_class(int64_t n) { return row_first_bitmap_class(n); }
int64_t bitmap_blocks(int64_t rows, int32_t r) { return row_bitmap_blocks(rows, r); }
uint32_t sort_blocks(int64_t rows, int k) { return row_sort_blocks(rows, k); }
uint32_t short_grid(uint32_t blocks) { return row_short_grid(blocks); }
int classes() { return kSortClasses; } int long_classes() { return kSortLongClasses; }
int k8k() { return kRow8k; } int k32k() { return kRow32k; } int klarge() { return kRowLarge; }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("row_sort")
    src, so = str(d / "shim.cpp"), str(d / "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_1606_07550_amd", "csrc"),
                    src, "-o", so], check=True)
    L = ctypes.CDLL(so)
    for f in (L.ranges, L.bitmap_min, L.first_class):
        f.argtypes = [ctypes.c_int64]
    L.bitmap_blocks.argtypes, L.bitmap_blocks.restype = [ctypes.c_int64, ctypes.c_int32], ctypes.c_int64
    L.sort_blocks.argtypes, L.sort_blocks.restype = [ctypes.c_int64, ctypes.c_int], ctypes.c_uint32
    L.short_grid.argtypes, L.short_grid.restype = [ctypes.c_uint32], ctypes.c_uint32
    return L


SIZES = sorted({1, 2, 1000, MOST_NODES} | {(1 << b) + d for b in range(16, 31) for d in (-1, 0, 1)}
               | {(k << 20) + d for k in (2, 3, 15, 16, 17, 31, 32, 33, 96, 129, 2047) for d in (-1, 0, 1)})


@pytest.mark.parametrize("n", SIZES)
def test_bitmap_launches_stay_in_the_limits(rules, n):
    r = rules.ranges(n)
    least = {rules.k8k(): 4097, rules.k32k(): 16385, rules.klarge(): max(32769, rules.bitmap_min(n))}
    first = rules.first_class(n)
    shortest = least[first]
    assert r == -(-n // (1 << 20))
    assert shortest >= rules.bitmap_min(n) or r == 1
    assert r == 1 or shortest >= 1024 * r  # work follows the entries, not the ids
    rows = min(n, MOST_ENTRIES // shortest)
    assert rules.bitmap_blocks(rows, r) >= rows * r
    assert rules.bitmap_blocks(rows, r) * 1024 < MOST_THREADS
    assert rows * r < 1 << 31 and rows * r * 256 < MOST_THREADS
    assert r == 1 or 8 * rows * r <= 4 * (MOST_ENTRIES // 2)  # two int32 each in m_raw int32


SHORTEST = [1025, 513, 257, 129, 65, 33, 17, 9, 2]  # entries of a row, by class from kRow4k down


@pytest.mark.parametrize("mix", [{k: 1.0} for k in range(9)] + [{8: 0.5, 5: 0.5}, {8: 0.45, 4: 0.55}, {0: 0.5, 2: 0.5},
                                                               {k: 1 / 9 for k in range(9)}])
def test_joint_launches_stay_in_the_limits(rules, mix):
    """The most rows that 2^31 entries make, of one class and of several."""
    assert rules.classes() == len(SHORTEST)
    blocks = [0, 0]
    for k, share in mix.items():
        rows = min(MOST_NODES, int(MOST_ENTRIES * share) // SHORTEST[k])
        blocks[k >= rules.long_classes()] += rules.sort_blocks(rows, k)
    assert max(blocks) < 1 << 32  # counted in 32 bits
    assert blocks[0] * 256 < MOST_THREADS
    assert rules.short_grid(blocks[1]) * 256 < MOST_THREADS
    assert rules.short_grid(1000) == 1000
