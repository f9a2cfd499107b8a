"""The rule that gives the even/odd block solver to the vector or to the matrix-core kernel
(csrc/sap_rule.h, plain C++), compiled with the host compiler and held against half-sweeps timed
on an MI355X with 256 CUs (BF16 storage, 4 MR steps): for each block shape the timed cases nearest
the rule's line on either side, among those where the two kernels differ by 4 % or more."""
import math
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MEASURED = {  # block: (blocks of a colour, rhs, us on the vector kernel, us on the matrix cores)
    (4, 4, 4, 4): [(1152, 3, 349, 322), (648, 9, 546, 504), (648, 5, 318, 365), (648, 2, 139, 174)],
    (8, 8, 2, 2): [(1152, 2, 377, 328), (648, 2, 236, 185)],
    (3, 5, 3, 5): [(648, 6, 401, 370), (432, 9, 394, 364), (432, 5, 221, 230), (648, 5, 328, 359)],
    (4, 4, 4, 3): [(1152, 3, 336, 310), (648, 9, 524, 493), (648, 5, 295, 354), (648, 2, 134, 170)],
    (7, 3, 3, 3): [(1152, 3, 342, 316), (648, 9, 542, 501), (192, 9, 163, 177), (432, 5, 211, 232)],
    (4, 5, 3, 3): [(1152, 3, 333, 312), (648, 9, 526, 497), (648, 5, 292, 354), (648, 2, 134, 172)],
    (3, 3, 3, 6): [(1152, 3, 318, 288), (256, 5, 118, 112), (192, 9, 155, 163), (432, 5, 203, 214)],
    (4, 4, 3, 3): [(1152, 3, 305, 292), (648, 9, 499, 466), (648, 5, 284, 334), (648, 2, 130, 166)],
    (6, 6, 2, 2): [(1152, 3, 310, 294), (128, 9, 117, 113), (192, 9, 155, 168), (432, 5, 201, 222)],
    (3, 3, 3, 5): [(1152, 3, 305, 290), (648, 9, 496, 461), (648, 5, 282, 331), (648, 2, 130, 165)],
    (1, 4, 8, 4): [(1152, 5, 455, 410), (648, 6, 296, 263), (192, 9, 118, 132), (192, 5, 81, 88)],
    (2, 2, 2, 16): [(1152, 5, 457, 408), (648, 6, 298, 260), (192, 9, 118, 130), (192, 5, 81, 88)],
    (2, 4, 4, 4): [(1152, 2, 170, 150), (648, 5, 255, 172), (648, 2, 89, 98)],
    (4, 4, 4, 2): [(1152, 2, 170, 152), (192, 9, 117, 99), (648, 2, 91, 98)],
    (8, 4, 2, 2): [(1152, 5, 470, 411), (648, 6, 309, 263), (192, 9, 122, 131), (192, 5, 83, 88)],
    (3, 2, 3, 7): [(1152, 5, 476, 412), (648, 6, 305, 262), (192, 9, 122, 132), (192, 5, 84, 88)],
    (1, 5, 5, 5): [(1152, 5, 476, 414), (648, 6, 312, 262), (192, 9, 123, 132), (192, 5, 85, 88)],
    (5, 5, 5, 1): [(256, 3, 50, 48), (192, 8, 97, 92), (192, 9, 123, 133), (432, 2, 85, 89)],
    (2, 3, 5, 4): [(1152, 2, 174, 151), (648, 5, 262, 172), (648, 2, 92, 99)],
    (3, 3, 3, 4): [(648, 6, 184, 175), (432, 9, 183, 174), (648, 5, 158, 172), (648, 3, 95, 101)],
    (4, 3, 3, 3): [(1152, 5, 281, 265), (648, 6, 184, 174), (648, 5, 159, 173), (648, 3, 95, 101)],
    (4, 5, 1, 5): [(1152, 2, 177, 149), (192, 9, 121, 98), (648, 2, 92, 98)],
    (5, 5, 2, 2): [(648, 6, 184, 172), (432, 9, 187, 175), (648, 5, 163, 172), (192, 9, 92, 99)],
    (2, 2, 2, 12): [(1152, 5, 269, 255), (648, 6, 181, 166), (648, 5, 156, 165), (192, 9, 90, 95)],
    (2, 2, 4, 6): [(1152, 5, 265, 253), (648, 6, 178, 167), (648, 5, 155, 165), (648, 3, 92, 96)],
    (2, 4, 4, 3): [(648, 6, 177, 166), (432, 9, 178, 165), (648, 5, 153, 165), (192, 9, 88, 94)],
    (2, 3, 3, 5): [(1152, 5, 263, 250), (648, 6, 180, 167), (648, 5, 155, 165), (192, 9, 88, 95)],
    (3, 3, 3, 3): [(1152, 5, 266, 247), (648, 6, 181, 166), (648, 5, 156, 165), (1152, 2, 121, 143)],
    (3, 3, 2, 4): [(1152, 5, 263, 243), (648, 6, 179, 163), (648, 5, 155, 162), (192, 9, 89, 93)],
    (1, 2, 5, 7): [(648, 6, 176, 166), (432, 9, 175, 165), (648, 5, 152, 164), (648, 3, 90, 95)],
    (1, 1, 8, 8): [(1152, 9, 408, 389), (192, 12, 111, 100), (432, 9, 150, 166), (648, 6, 151, 168)],
    (1, 4, 4, 4): [(432, 5, 112, 93), (432, 6, 113, 94), (128, 8, 41, 44), (256, 4, 41, 44)],
    (2, 2, 2, 8): [(432, 5, 111, 93), (432, 6, 113, 93), (128, 8, 41, 44), (256, 4, 41, 44)],
    (4, 4, 2, 2): [(1152, 2, 114, 109), (648, 5, 148, 115), (128, 8, 41, 43), (256, 4, 41, 44)],
    (4, 4, 4, 1): [(1152, 2, 117, 111), (432, 5, 115, 92), (128, 5, 40, 42), (128, 6, 40, 42)],
    (3, 3, 3, 2): [(1152, 2, 117, 95), (648, 5, 153, 111), (128, 5, 40, 42), (128, 6, 40, 42)],
    (2, 2, 2, 6): [(1152, 2, 117, 93), (648, 5, 153, 106), (128, 8, 41, 43), (128, 5, 39, 41)],
    (1, 3, 3, 5): [(1152, 2, 116, 94), (648, 5, 151, 107), (128, 8, 42, 43), (256, 4, 42, 43)],
    (2, 2, 3, 3): [(1152, 2, 112, 87), (648, 5, 146, 101), (192, 5, 40, 51), (432, 2, 39, 52)],
    (3, 3, 2, 2): [(1152, 2, 112, 87), (648, 5, 147, 98)],
    (2, 4, 2, 2): [(648, 2, 73, 43), (256, 5, 72, 42), (192, 5, 38, 41), (432, 2, 38, 41)],
    (2, 2, 2, 3): [(648, 2, 76, 43), (256, 5, 72, 41)],
    (2, 2, 2, 2): [(648, 2, 73, 38), (256, 5, 69, 38)],
    (1, 1, 1, 8): [(648, 2, 59, 38), (256, 5, 57, 38), (128, 8, 32, 36), (256, 4, 32, 36)],
    (1, 2, 2, 2): [(648, 2, 74, 38), (256, 5, 72, 37)],
}

PROGRAM = r"""
#include <cstddef>
#include <cstdio>
#include "sap_rule.h"
int main() {
  const size_t lds = 160 * 1024;
  int bv, entries, blocks, rhs, per_item;
  while (std::scanf("%d %d %d %d %d", &bv, &entries, &blocks, &rhs, &per_item) == 5) {
    const size_t half = (bv + 1) / 2, slots = 2 * half + 1, e = entries;
    // exchange rows, border entries and links as the kernels lay them out
    const size_t vec = 96 + 96 * 2 * half + 96 * e;
    const size_t xch = slots * 448 > e * 192 ? slots * 448 : e * 192;
    const size_t mm = xch + (4 * slots * 36 + 15) / 16 * 16 + 512 + 4 * slots;
    std::printf("%d\n", (int)wc::sap_mm_faster((long long)blocks * rhs, int(2 * half + 63) / 64, vec,
                                               (long long)blocks * ((rhs + per_item - 1) / per_item),
                                               int(half + 15) / 16, mm, lds, 256));
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("rule")
    (d / "rule.cpp").write_text(PROGRAM)
    cc = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I",
                         os.path.join(ROOT, "paper_1109_4279_amd", "csrc"), str(d / "rule.cpp"), "-o", str(d / "rule")],
                        capture_output=True, text=True, timeout=120)
    assert cc.returncode == 0, cc.stderr

    def picks(cases):
        """cases of (block, blocks, rhs, rhs per matrix-core item) -> whether on the matrix cores"""
        lines = []
        for block, blocks, rhs, per_item in cases:
            bv = math.prod(block)
            lines.append(f"{bv} {sum(2 * bv // b for b in block)} {blocks} {rhs} {per_item}")
        run = subprocess.run([str(d / "rule")], input="\n".join(lines), capture_output=True, text=True, timeout=120)
        assert run.returncode == 0
        return [bool(int(v)) for v in run.stdout.split()]

    return picks


def test_pick_is_the_faster_kernel(rule):
    cases = [(b, blocks, rhs, vec, mm) for b, rows in MEASURED.items() for blocks, rhs, vec, mm in rows]
    got = rule([(b, blocks, rhs, 4) for b, blocks, rhs, _, _ in cases])
    assert len(got) == len(cases)
    wrong = [c for c, g in zip(cases, got) if g != (c[4] < c[3])]
    assert not wrong, wrong


def test_few_items_and_large_blocks_stay_on_the_vector_kernel(rule):
    """Up to two items per CU; a block whose faces do not fit the LDS; one rhs per item."""
    assert rule([((4, 4, 4, 4), 256, 2, 4), ((2, 2, 2, 2), 128, 4, 4)]) == [False, False]
    assert rule([((1, 1, 1, 256), 1000, 12, 4), ((2, 2, 2, 32), 1000, 12, 4)]) == [False, False]
    assert not any(rule([(b, 4000, 1, 1) for b in ((4, 4, 4, 4), (4, 3, 3, 3), (4, 4, 2, 2))]))


def test_more_right_hand_sides_in_a_tile_never_lose_it(rule):
    """From a tile of two to a full one the matrix cores' time stays and the vector kernel's
    grows: once picked, picked."""
    for b in MEASURED:
        for blocks in (64, 200, 256, 300, 700, 2000, 10000):
            got = rule([(b, blocks, n, 4) for n in (2, 3, 4)])
            assert got == sorted(got), (b, blocks, got)
