"""The byte ranges that the ring kernel's loads of rows in phases may touch
(csrc/ragged_rows.hpp, compiled here): every row of the block, and at most the
rest of the dword that holds the block's last byte."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# the kernel's steps (xcorr16.hpp: wave_main), for every phase and stage
PROGRAM = r"""
#include <cstdio>
#include <cstdint>
#include <initializer_list>
#include <numeric>
#include "ragged_rows.hpp"
using namespace xeng::x16;
int main() {
  long checked = 0;
  for (int unit : {4, 16})
    for (int n = 1; n <= 40; ++n)
      for (int f = 1; f <= 9; ++f)
        for (int T : {1, 2, 3, 15, 16, 17, 63, 64, 65, 130, 1025}) {
          const uint32_t row = f * n;
          const int period = unit / std::gcd(row, (uint32_t)unit);
          const uint32_t stride = period * row;
          const uint64_t size = (uint64_t)T * row, end = (size + 3) & ~3ull;
          for (int phase = 0; phase < period && phase < T; ++phase) {
            const uint64_t off = (uint64_t)phase * row;
            const uint32_t sub = off & (unit - 1), slack = row_slack(stride, sub, row);
            const int rows_all = (T - phase + period - 1) / period;
            for (int first = 0; first < rows_all; first += 64, ++checked) {
              const int rows = rows_all - first < 64 ? rows_all - first : 64;
              const uint64_t base = off - sub + (uint64_t)first * stride;
              const uint64_t limit = base + stage_bytes(rows, stride, slack);
              const uint64_t last = off + (uint64_t)(first + rows - 1) * stride + row;
              if (stride % unit || limit > end || limit < last || (limit - base) % 4) {
                printf("unit %d n %d f %d T %d phase %d first %d: %llu of %llu\n", unit, n, f, T, phase, first,
                       (unsigned long long)limit, (unsigned long long)size);
                return 1;
              }
            }
          }
        }
  static_assert(stage_bytes(0, 160, 8) == 0, "a stage past the range reads nothing");
  printf("%ld\n", checked);
}
"""


def test_loads_end_with_the_block(tmp_path):
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(PROGRAM)
    cmd = ["g++", "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "paper_1904_07778_amd", "csrc"), str(src), "-o", str(exe)]
    try:
        subprocess.run(cmd, check=True, capture_output=True, text=True)
    except FileNotFoundError:
        pytest.skip("no g++")
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout) > 10000
