"""The scatter's map from blocks to slots and groups, compiled for the host: every group of every slot is taken by
exactly one block, and the eight XCDs (block b runs on XCD b mod 8) get the same number of working blocks, within one,
also where there are fewer slots than XCDs or a few more."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_07387_amd", "csrc")
PROGRAM = r"""
#include "block_map.h"
#include <algorithm>
#include <cstdio>
#include <vector>
int main() {
  for (uint32_t n : {1u, 2u, 3u, 5u, 7u, 8u, 9u, 12u, 15u, 16u, 17u, 31u, 100u, 1001u})
    for (uint32_t gx : {1u, 2u, 3u, 7u, 8u, 9u, 64u, 1023u}) {
      std::vector<int> taken((size_t)n * gx, 0);
      uint32_t per[8] = {};
      const uint32_t blocks = tn::slot_blocks(n, gx);
      if (blocks % 8 != 0 || blocks < n * gx || blocks >= n * gx + 8) return std::printf("blocks %u %u\n", n, gx), 1;
      for (uint32_t b = 0; b < blocks; ++b) {
        const tn::SlotBlock s = tn::slot_block(b, n, gx);
        if (s.slot >= n) continue;
        if (s.group >= gx) return std::printf("group %u %u\n", n, gx), 1;
        ++taken[(size_t)s.slot * gx + s.group];
        ++per[b % 8];
      }
      if (std::any_of(taken.begin(), taken.end(), [](int t) { return t != 1; }))
        return std::printf("cover %u %u\n", n, gx), 1;
      if (*std::max_element(per, per + 8) - *std::min_element(per, per + 8) > 1)
        return std::printf("balance %u %u\n", n, gx), 1;
    }
  return 0;
}
"""


def test_map(tmp_path):
    src, exe = tmp_path / "map.cpp", tmp_path / "map"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(exe), str(src)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
