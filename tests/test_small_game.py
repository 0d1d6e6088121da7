"""Shares of the threads in the Gram matrix of a game of at most 64 players (csrc/small_game.h), compiled for the host:
every pair of players is stored by one thread of a workgroup, and every row adds to it once."""
import os
import shutil
import subprocess


ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAIN = r"""
#include <stdio.h>
#include "small_game.h"
int main() {   // players, pair, threads that store it, threads that add the rows of each group to it (least and most)
  for (int n = 1; n <= kSmallMax; ++n) {
    const int pairs = n * (n + 1) / 2;
    for (int p = 0; p < pairs; ++p) {
      int stores = 0, adds[kSmallThreads] = {0}, groups = 0;
      for (int tid = 0; tid < kSmallThreads; ++tid) {
        const ds_small_share s = ds_small_share_of(pairs, tid);
        groups = s.groups;
        for (int u = 0; u < kSmallPerThread; ++u) {
          if (s.at + u * s.width != p) continue;
          if (ds_small_stores(s)) ++stores;
          if (ds_small_adds(s)) ++adds[s.group];
        }
      }
      int least = adds[0], most = adds[0];
      for (int g = 1; g < groups; ++g) {
        least = adds[g] < least ? adds[g] : least;
        most = adds[g] > most ? adds[g] : most;
      }
      printf("%d %d %d %d %d\n", n, p, stores, least, most);
    }
  }
  return 0;
}
"""


def test_every_pair_has_one_writer(tmp_path):
    cxx = shutil.which("g++") or "/opt/rocm/bin/amdclang++"
    src = tmp_path / "main.cpp"
    src.write_text(MAIN)
    subprocess.run([cxx, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2506_22668_amd", "csrc"), str(src),
                    "-o", str(tmp_path / "main")], check=True)
    out = subprocess.run([str(tmp_path / "main")], capture_output=True, text=True, check=True).stdout.split("\n")
    rows = [tuple(map(int, line.split())) for line in out if line]
    assert len(rows) == sum(n * (n + 1) // 2 for n in range(1, 65))
    wrong = sorted({n for n, _, stores, least, most in rows if (stores, least, most) != (1, 1, 1)})
    assert not wrong, f"games of {wrong} players"
