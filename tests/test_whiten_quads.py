"""Which positions a wave of the whitening reads at a row's ends: the rule that the kernel uses (csrc/espo_quad.h), compiled for
the host.  No position outside of the row's valid span may be read, and each one inside belongs to exactly one lane."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "espo_quad.h"
int main() {
  for (int lo = 0; lo < 4; ++lo)
    for (int hi = 0; hi <= 1024; hi += hi < 24 || hi > 1000 ? 1 : 13) {  // an item: 1024 positions, a span of them valid
      std::vector<int> owned(1024 + 8, 0);
      for (int t = 0; t < 1024; t += 4) {
        const espo::Quad q = espo::quad_of(t, lo, hi);
        for (int j = 0; j < 4; ++j) {
          const bool own = (q.in >> j) & 1u, read = hi - lo >= 4 ? q.in != 0 : own;
          const int p = q.at + j;
          if (read && (p < lo || p >= hi)) return std::printf("t=%d span [%d, %d): reads %d\n", t, lo, hi, p), 1;
          if (own && (p < t || p >= t + 4)) return std::printf("t=%d span [%d, %d): owns %d\n", t, lo, hi, p), 1;
          if (own) ++owned[p];
        }
        if (q.in > 0xfu || (q.in == 0xfu && q.at != t)) return std::printf("t=%d span [%d, %d): whole but moved\n", t, lo, hi), 1;
      }
      for (int p = 0; p < (int)owned.size(); ++p)
        if (owned[p] != (p >= lo && p < hi)) return std::printf("span [%d, %d): %d owners of %d\n", lo, hi, owned[p], p), 1;
    }
  return 0;
}
"""


def test_only_valid_positions_are_read_and_each_by_its_owner(tmp_path):
    src, exe = tmp_path / "quads.cpp", tmp_path / "quads"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
                    "-I" + os.path.join(ROOT, "paper_2605_29860_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
