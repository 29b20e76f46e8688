"""Which query blocks go in pairs and which pairs are left over (csrc/attn_pairs.h), on the host: every block in one slot and one pair, fewer than a
round of pairs left, no text among them, for all lengths from 505 blocks to 1 200."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "attn_pairs.h"
using namespace dfs;
static int check(int M_v, int M_x, int heads) {
  const int M = M_v + M_x, slots = pair_slots(M_v, M, heads), rounds = slots / PAIR_WGS;
  std::vector<char> taken(size_t(heads) * M, 0);
  for (int slot = 0; slot < slots; ++slot)
    for (int xcd = 0; xcd < 8; ++xcd) {
      int head;
      const int u = pair_at(xcd, slot, M_v, M, heads, head), end = u < M_v ? M_v : M;
      if (u < 0) continue;
      if (u >= end || head < 0 || head >= heads) return 1;
      if (u >= M_v && slot >= rounds * PAIR_WGS) return 2;
      for (int b = u; b < u + 2 && b < end; ++b) {
        if (taken[size_t(head) * M + b]++) return 3;
        if (pair_of(b, M_v) != u || pair_slot(head, b, M_v, M, heads) != slot) return 4;
      }
    }
  for (char t : taken)
    if (!t) return 5;
  return slots - rounds * PAIR_WGS >= PAIR_WGS ? 6 : 0;
}
int main() {
  for (int M_v = 505; M_v <= 1200; ++M_v)
    for (int heads = 1; heads <= 48; heads += heads < 6 ? 1 : 7)
      for (int M_x : {0, 1, 2, 5})
        if (int e = check(M_v, M_x, heads)) return std::printf("%d + %d blocks x %d heads: %d\n", M_v, M_x, heads, e), 1;
  return check(513, 4000, 2) || check(4096, 0, 2) || check(65535, 1, 1);
}
"""


def test_every_block_is_in_one_pair(tmp_path):
    cxx = shutil.which("g++") or pytest.skip("no host compiler")
    (tmp_path / "rules.cpp").write_text(PROGRAM)
    subprocess.run([cxx, "-O2", "-std=c++17", "-D__host__=", "-D__device__=", "-D__forceinline__=inline", "-I", os.path.join(ROOT, "paper_2605_23445_amd", "csrc"),
                    str(tmp_path / "rules.cpp"), "-o", str(tmp_path / "rules")], check=True)
    done = subprocess.run([str(tmp_path / "rules")], capture_output=True, text=True)
    assert done.returncode == 0, done.stdout
