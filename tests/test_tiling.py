"""The video kernel's tiling rule (ws_kernels.hpp: video_tiling), on the CPU,
compiled with the host compiler.

- video_group_count looks at the counts that can be cheapest only; over a grid
  it picks what a scan of every count picks.
- A narrower query tile never takes more key ranges per head than the full one
  (so a call that fits the split-KV workspace still fits), nor more heads per
  workgroup where the full one takes one each, and its waves cover the rows.
- The picks for the shapes whose times the rule's comment gives."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_04443_amd", "csrc")

PROGRAM = r"""
#include "ws_kernels.hpp"
#include <cstdio>

static long long scan(long long heads, long long qtiles, long long pages, long long cus) {
  if (pages == 0) return heads;
  const long long units = heads * pages, round = cus / qtiles > 1 ? cus / qtiles : 1;
  long long top = heads * (ws::kMaxVideoSplits - 1);
  if (units < top) top = units;
  if (4 * round < top) top = 4 * round;
  long long best = heads < top ? heads : top;
  double best_cost = -1;
  for (long long g = 1; g <= top; ++g) {
    const bool whole = g % heads == 0 || heads % g == 0;
    const double segs = (double)(whole ? (g > heads ? g : heads) : g + heads - 1) / g;
    const double cost = (double)((g + round - 1) / round) * ((double)units / g + 9.5 * segs) +
                        (ws::video_heads_split(heads, g) ? 4.0 : 0.0);
    if (best_cost < 0 || cost < best_cost - 1e-9) { best = g; best_cost = cost; }
  }
  return best;
}

int main() {
  long long n = 0;
  for (int h = 1; h <= 64; ++h)
    for (int qt : {1, 2, 3, 4, 5, 8, 17})
      for (int p : {0, 1, 2, 5, 13, 19, 38, 49, 139, 479, 5000})
        for (int cus : {1, 4, 85, 256}) {
          if (scan(h, qt, p, cus) != ws::video_group_count(h, qt, p, cus)) {
            std::printf("FAIL count h=%d qt=%d p=%d cus=%d\n", h, qt, p, cus);
            return 1;
          }
          ++n;
        }
  for (int h : {1, 3, 12, 17, 40, 64})
    for (int q = 1; q <= 1100; q += 13)
      for (int p : {0, 1, 5, 13, 38, 139, 479})
        for (int cus : {4, 85, 256}) {
          const ws::VideoTiling t = ws::video_tiling(h, q, p, cus);
          const long long wide = ws::video_group_count(h, (q + 255) / 256, p, cus);
          const bool known = t.rows == 256 || t.rows == 192 || t.rows == 128;
          if (!known || (q <= 128 && t.rows != 256) || t.groups < 1 ||
              t.groups != ws::video_group_count(h, (q + t.rows - 1) / t.rows, p, cus) ||
              ws::video_max_ranges(h, t.groups) > ws::video_max_ranges(h, wide) ||
              (wide == h && h * ((q + 255) / 256) <= cus && t.groups < h)) {
            std::printf("FAIL tiling h=%d q=%d p=%d cus=%d rows=%d groups=%lld\n", h, q, p, cus, t.rows, (long long)t.groups);
            return 1;
          }
          // the waves of a tile cover its rows, whatever part of it is used
          for (int rows = 1; rows <= t.rows; ++rows)
            if (ws::kVideoWaves * ws::video_wave_rows(t.rows, rows) < rows) { std::printf("FAIL cover\n"); return 1; }
          ++n;
        }
  struct { int h, q, p, rows, groups; } pinned[] = {{12, 252, 13, 192, 84}, {40, 920, 19, 192, 40}, {17, 333, 38, 128, 85},
                                                    {40, 920, 49, 192, 40}, {40, 920, 139, 256, 64}, {40, 920, 479, 256, 64},
                                                    {3, 129, 5, 128, 3}, {3, 250, 5, 192, 3}, {3, 500, 5, 192, 3}, {3, 380, 5, 256, 3}, {3, 300, 5, 128, 3},
                                                    {24, 2048, 1, 256, 24}, {28, 1784, 2, 256, 28}, {64, 1024, 2, 256, 64}, {46, 1016, 2, 256, 46}};
  for (auto& c : pinned) {
    const ws::VideoTiling t = ws::video_tiling(c.h, c.q, c.p, 256);
    if (t.rows != c.rows) { std::printf("FAIL pinned h=%d q=%d p=%d: %d\n", c.h, c.q, c.p, t.rows); return 1; }
    if (c.h > 3 && t.groups != c.groups) { std::printf("FAIL groups h=%d: %lld\n", c.h, (long long)t.groups); return 1; }
  }
  std::printf("ok %lld\n", n);
  return 0;
}
"""


def test_tiling_rule(tmp_path):
    src, exe = tmp_path / "tiling.cpp", tmp_path / "tiling"
    src.write_text(PROGRAM)
    try:
        subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                        "-I", CSRC, str(src), "-o", str(exe)], check=True, capture_output=True, text=True)
    except FileNotFoundError:
        pytest.skip("no host C++ compiler")
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
    assert out.stdout.startswith("ok")
