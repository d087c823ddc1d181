"""The expansion kernel's LDS layout (csrc/kernels.h), on the host: every tree
shape that s2moe_expand accepts has room for the bitsets of all its nodes."""

import subprocess

from paper_2608_15018_amd import build as B

SOURCE = r"""
#include <cstdio>
#include "kernels.h"
using namespace s2moe;
int main() {
  // A bitset has w = 1, 2, 4, ... 32 words, whatever E rounds up to 32 w and
  // whatever k is.
  long shapes = 0;
  for (int w = 1; w <= 32; w <<= 1)
    for (int L = 1; L <= 128; ++L)
      for (int N = 1; N <= 1024; ++N) {
        const size_t accepted = expand_accept_bytes(N, L, 32 * w);
        const ExpandLds o = expand_lds(N, L, 32 * w, N, 1);
        const size_t row = (size_t)L * w * 4;
        if (o.total > accepted || o.rows % 16 || (w >= 4 && (row % 16 || o.uni % 16)) ||
            (w == 2 && o.uni % 8) || o.pv % 8 || o.cdr % 4 || o.rows + N * row > o.uni ||
            o.uni + row > o.pv || o.pv + 8 * N > o.cdr || o.cdr + 4 * N > o.node ||
            o.node + 2 * N > o.list || o.list + 2 * N > o.total) {
          std::printf("N = %d, L = %d, %d words: %zu bytes for %zu\n", N, L, w, o.total, accepted);
          return 1;
        }
        ++shapes;
      }
  std::printf("%ld\n", shapes);
}
"""


def test_all_bitsets_fit_every_accepted_shape(tmp_path):
    src, exe = tmp_path / "lds.cpp", tmp_path / "lds"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__=1", "-I", B.ROCM_INC,
                    "-I", B.CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout) == 6 * 128 * 1024
