"""Cuts of the matrix-core product into workgroups (csrc/mm_split.h), compiled for the host: the chosen cuts of measured
shapes, the bounds of the column groups, and the shares of an even cut."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHUNK, ROWS, MAX_CPG = 1024, 256, 1024

# what the library asks for: sums priced at 32 bytes a row for the column groups, at 16 for the even cut
MAIN = r"""
#include <stdio.h>
#include <string.h>
#include <vector>
#include "mm_split.h"
int main() {
  long long cus, r, c;
  while (scanf("%lld %lld %lld", &cus, &r, &c) == 3) {
    const int64_t rg = (r + @ROWS@ - 1) / @ROWS@, nc = (c + @CHUNK@ - 1) / @CHUNK@;
    const ds_mm_split s = ds_mm_choose_split(cus, r, rg, nc, @MAX_CPG@, 32);
    ds_mm_even e = ds_mm_choose_even(cus, r, rg, nc, @MAX_CPG@, 16, s);
    const long long chosen = e.wgs;
    if (e.wgs == 0) {   // its shares are looked at all the same, if it could be taken
      ds_mm_split dear = {nc * 100000, 100000};
      e = ds_mm_choose_even(cus, r, rg, nc, @MAX_CPG@, 16, dear);
    }
    // as bit_spmv_mm_kernel walks them: units, each once; sums, each slot of a row group once; chunks of a row group in one sum
    const int64_t units = rg * nc;
    long long shares = 0, twice = 0, outside = 0, empty = 0, longest = 0, next = 0;
    std::vector<char> taken((size_t)(rg * (e.slots > 0 ? e.slots : 1)), 0);
    for (int64_t b = 0; b < e.wgs; ++b) {
      const int64_t u0 = ds_mm_even_begin(b, e.wgs, units);
      int64_t left = ds_mm_even_begin(b + 1, e.wgs, units) - u0, g = u0 / nc, ch = u0 - g * nc;
      int64_t slot = b - ds_mm_even_owner(g * nc, e.wgs, units);
      empty += left < 1;
      shares += u0 == next ? left : 0;
      next = u0 + left;
      for (long long run = 0; left > 0; --left) {
        ++run;
        longest = run > longest ? run : longest;
        if (ch == nc - 1 || left == 1) {
          if (slot < 0 || slot >= e.slots || g >= rg) ++outside;
          else twice += taken[(size_t)(g * e.slots + slot)]++;
          slot = 0;
          run = 0;
        }
        if (++ch == nc) ch = 0, ++g;
      }
    }
    printf("%lld %lld %lld %lld %lld %lld %lld %lld %lld %lld\n", (long long)s.cpg, (long long)s.groups, chosen, (long long)e.wgs,
           shares == units, (long long)(next == units), twice, outside, empty, longest);
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    cxx = shutil.which("g++") or "/opt/rocm/bin/amdclang++"
    d = tmp_path_factory.mktemp("mm_split")
    src = d / "main.cpp"
    src.write_text(MAIN.replace("@ROWS@", str(ROWS)).replace("@CHUNK@", str(CHUNK)).replace("@MAX_CPG@", str(MAX_CPG)))
    subprocess.run([cxx, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2506_22668_amd", "csrc"), str(src),
                    "-o", str(d / "main")], check=True)

    def run(shapes):
        text = "\n".join(" ".join(map(str, s if len(s) == 3 else (256, *s))) for s in shapes)
        out = subprocess.run([str(d / "main")], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        keys = ("cpg", "groups", "even", "wgs", "whole", "ends", "twice", "outside", "empty", "longest")
        return [dict(zip(keys, map(int, line.split()))) for line in out if line]
    return run


# (rows, columns): us of a CGLS iteration by the cut of this product, the even one (0) or a number of column groups, the other
# product as chosen
MEASURED = {
    (34177, 99981): {0: 275.8, 1: 331.8, 3: 290.4, 5: 284.8, 7: 282.7, 8: 285.7, 11: 283.0, 20: 283.1, 33: 290.0},
    (99981, 34177): {0: 275.5, 1: 285.1, 3: 276.7, 4: 280.8, 5: 278.8, 8: 279.2, 16: 283.8},
    (10253, 99981): {0: 116.3, 1: 231.5, 5: 120.2, 6: 117.2, 10: 120.0, 11: 117.5, 13: 116.5, 25: 118.8},
    (9410, 300007): {0: 248.6, 5: 266.4, 6: 254.5, 11: 258.0, 13: 253.3, 20: 250.6, 33: 253.5},
    (300007, 9410): {0: 248.5, 1: 245.4, 2: 249.5, 3: 249.7, 4: 253.8},
    (32347, 200003): {0: 457.9, 2: 452.3, 3: 493.9, 4: 456.1, 6: 459.0, 8: 460.2, 16: 470.9},
    (200003, 32347): {0: 458.1, 1: 512.3, 2: 495.0, 3: 496.3, 5: 493.3, 8: 503.4},
    (500009, 15102): {0: 561.5, 1: 542.0, 2: 554.2, 3: 557.3, 5: 564.6},   # one column group is 3.5 % faster
    (18111, 50021): {0: 105.3, 1: 152.4, 3: 108.1, 5: 111.7, 7: 105.0, 8: 104.9, 16: 109.2},
    (50021, 18111): {0: 105.2, 1: 109.2, 2: 107.3, 4: 107.9, 8: 107.4},
    (7857, 20011): {0: 63.3, 1: 84.1, 3: 65.8, 5: 62.3, 7: 61.7, 8: 61.7, 10: 63.4, 16: 63.4},
    (20011, 7857): {0: 62.4, 1: 68.4, 2: 62.2, 3: 61.7, 4: 63.2, 8: 63.1},
    (3414, 100428): {0: 75.3, 5: 92.3, 10: 78.9, 16: 75.5, 20: 78.6, 33: 76.4},
    (100428, 3414): {0: 75.4, 1: 73.8, 2: 76.9, 4: 80.2},                  # 2 %
    (628, 300007): {0: 72.6, 16: 92.1, 33: 77.9, 48: 75.6, 74: 71.3},
    (4244, 9000): {0: 62.3, 1: 73.3, 3: 64.7, 5: 63.5, 9: 62.1},
}


def test_measured_shapes_take_a_fast_cut(cut):
    for (shape, us), c in zip(MEASURED.items(), cut(MEASURED)):
        chosen = 0 if c["even"] else c["groups"]
        limit = {(500009, 15102): 1.04, (100428, 3414): 1.03}.get(shape, 1.015)
        assert us[chosen] <= limit * min(us.values()), (shape, chosen)


def test_every_split_covers_the_columns(cut):
    shapes = [(1, 1), (1, 1024), (255, 1025), (256, 4096), (257, 1 << 20), (131072, 4097), (131073, 2049),
              (1, (1 << 22) + 5), (500000, 1 << 21), (3, 10 ** 7)]
    for (rows, cols), c in zip(shapes, cut(shapes)):
        chunks = -(-cols // CHUNK)
        cpg, groups = c["cpg"], c["groups"]
        assert 1 <= cpg <= MAX_CPG and (groups - 1) * cpg < chunks <= groups * cpg, (rows, cols, cpg, groups)


# one unit; fewer units than compute units, as many, one more; row groups of one chunk; a row group that many workgroups share; sums
# that would be longer than the accumulators hold (no even cut); a last row group and chunk that are not full
def test_shares_of_an_even_cut(cut):
    shapes = [(cus, rows, cols) for cus in (1, 3, 64, 255, 256, 304)
              for rows in (1, 256, 257, 255 * 256, 256 * 256, 256 * 257, 7857, 99981, 300007)
              for cols in (1, 1024, 1025, 20011, 255 * 1024, 256 * 1024, 256 * 1024 + 1)]
    shapes += [(256, 1, 1 << 28), (256, 300, (1 << 28) + 1), (256, 1000, 1 << 24), (1, 1, 1 << 20), (1, 1, (1 << 20) + 1)]
    none = 0
    for shape, c in zip(shapes, cut(shapes)):
        if c["wgs"] == 0:
            none += 1
            assert not c["even"]
            continue
        assert c["whole"] and c["ends"], shape
        assert (c["twice"], c["outside"], c["empty"]) == (0, 0, 0), (shape, c)
        assert c["longest"] <= MAX_CPG, (shape, c)
        assert c["wgs"] <= shape[0], shape
    assert none >= 1   # (1, (1 << 20) + 1) on one compute unit
