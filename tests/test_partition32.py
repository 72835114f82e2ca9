"""The attention kernel's form of the work partition (ws_kernels.hpp: FastDiv,
VideoPartition32), on the CPU: reciprocal divisions and 32-bit lookups give
the integers of plain division and of the 64-bit lookups, over ordinary
partitions, over ones whose products leave 32 bits, and at the divisors'
edges."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_04443_amd", "csrc")

PROGRAM = r"""
#include "ws_kernels.hpp"
#include <cstdio>

int main() {
  const unsigned top = 0x7fffffffu;
  for (unsigned d : {1u, 2u, 3u, 5u, 6u, 7u, 64u, 139u, 145u, 256u, 5800u, 65535u, 65536u, 65537u, 1000003u,
                     0x40000000u, 0x40000001u, 0x7ffffffeu, 0x7fffffffu}) {
    const ws::FastDiv f = ws::make_fast_div(d);
    for (unsigned k = 0; k < 4000; ++k)
      for (unsigned x : {k, top - k, k * d, k * d + d - 1, k * d + 1, k * 536870u, (top / d) * d - k}) {
        x &= top;
        if (ws::fast_div(x, f) != x / d) { std::printf("FAIL div %u / %u\n", x, d); return 1; }
      }
  }
  long long n = 0;
  for (long long heads : {1, 3, 12, 17, 40, 64, 4096})
    for (long long pages : {1, 2, 5, 13, 139, 499, 9000, 200000})
      for (long long cost : {0, 1, 6})
        for (long long groups : {1, 2, 7, 40, 63, 64, 84, 256, 480, 4096, 32768}) {
          if (groups > heads * pages || heads * pages > 9500000) continue;
          const ws::VideoPartition p{heads, pages, cost, groups};
          const ws::VideoPartition32 q = ws::make_part32(p);
          const long long gs = groups / 97 + 1, units = heads * pages, us = units / 997 + 1;
          for (long long g = 0; g <= groups; g += (groups - g > 3 ? gs : 1))
            if (ws::part_group_lo(q, g) != ws::video_group_lo_wide(p, g)) {
              std::printf("FAIL lo h=%lld p=%lld c=%lld G=%lld g=%lld\n", heads, pages, cost, groups, g);
              return 1;
            }
          for (long long x = 0; x < units; x += (units - x > 3 ? us : 1), ++n)
            if (ws::part_group_of(q, x) != ws::video_group_of_wide(p, x)) {
              std::printf("FAIL of h=%lld p=%lld c=%lld G=%lld x=%lld\n", heads, pages, cost, groups, x);
              return 1;
            }
        }
  std::printf("ok %lld\n", n);
  return 0;
}
"""


def test_partition32_equals_the_wide_lookups(tmp_path):
    src, exe = tmp_path / "part32.cpp", tmp_path / "part32"
    src.write_text(PROGRAM)
    try:
        subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                        "-I", CSRC, str(src), "-o", str(exe)], check=True, capture_output=True, text=True)
    except FileNotFoundError:
        pytest.skip("no host C++ compiler")
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
    assert out.stdout.startswith("ok")
