"""Work-group id -> (batch item, tile row, tile column) on the host: the
kernels' 32-bit arithmetic against plain 64-bit division, and every tile
visited once."""
import os
import subprocess

import pytest

SRC = r"""
#include <cstdio>
#include <vector>
#include "gemm_f32.hpp"
using namespace kt;
static bool reference(uint32_t pid, int tiles_m, int tiles_n, int64_t batch, int& tm, int& tn, int64_t& bz) {
  const int64_t nt = (int64_t)tiles_m * tiles_n, per = nt * batch / 8;
  int64_t t = pid;
  if (t < per * 8) t = (t % 8) * per + t / 8;
  bz = t / nt;
  t -= bz * nt;
  const int64_t width = (int64_t)8 * tiles_n, first = t / width * 8, r = t % width;
  const int64_t rows = tiles_m - first < 8 ? tiles_m - first : 8;
  tm = (int)(first + r % rows);
  tn = (int)(r / rows);
  return true;
}
static GemmArgs args(int tiles_m, int tiles_n, int64_t batch) {
  GemmArgs g{};
  set_geometry(g, tiles_m, tiles_n, batch);
  return g;
}
int main() {
  const uint32_t ds[] = {1, 2, 3, 5, 7, 8, 9, 63, 64, 65, 1000, 4095, 65537, 1u << 20, (1u << 26) - 1, 1u << 26,
                         0x7fffffffu, 0x80000000u, 0xfffffffeu, 0xffffffffu};
  for (uint32_t d : ds) {
    const FastDiv f = FastDiv::make(d);
    for (uint64_t k = 0; k < 4000; ++k) {
      const uint64_t base = k * 1073807u % 0x100000000ull + 1;
      for (int64_t e = -1; e <= 1; ++e) {
        for (uint64_t n : {(uint64_t)(base + e), (uint64_t)(base / d * d + e), (uint64_t)(0xffffffffu - k)}) {
          if (n > 0xffffffffull) continue;
          if (f((uint32_t)n) != (uint32_t)n / d) { printf("div %u / %u\n", (uint32_t)n, d); return 1; }
        }
      }
    }
  }
  for (int tm_n : {1, 2, 3, 7, 8, 9, 15, 16, 17, 40})
    for (int tn_n : {1, 2, 5, 8, 13, 33})
      for (int64_t batch : {1, 2, 3, 8, 31}) {
        const GemmArgs g = args(tm_n, tn_n, batch);
        const uint32_t total = (uint32_t)(tm_n * tn_n * batch);
        std::vector<int> seen(total, 0);
        for (uint32_t p = 0; p < total; ++p) {
          int tm, tn, rm, rn;
          int64_t b, rb;
          block_coords(p, g, tm, tn, b);
          reference(p, tm_n, tn_n, batch, rm, rn, rb);
          if (tm != rm || tn != rn || b != rb || tm < 0 || tm >= tm_n || tn < 0 || tn >= tn_n) {
            printf("block %u of %d x %d x %d\n", p, tm_n, tn_n, (int)batch);
            return 1;
          }
          ++seen[(b * tm_n + tm) * tn_n + tn];
        }
        for (int v : seen) if (v != 1) { printf("tile missed\n"); return 1; }
      }
  // the largest grids: 2^26 work-groups, one row or one column of tiles
  const int big[][2] = {{1, 1 << 26}, {1 << 26, 1}, {8191, 8192}, {(1 << 26) - 1, 1}};
  for (auto& s : big) {
    const GemmArgs g = args(s[0], s[1], 1);
    for (uint32_t k = 0; k < 200000; ++k) {
      const uint32_t p = (uint32_t)((uint64_t)k * 1000003u % ((uint64_t)s[0] * s[1]));
      int tm, tn, rm, rn;
      int64_t b, rb;
      block_coords(p, g, tm, tn, b);
      reference(p, s[0], s[1], 1, rm, rn, rb);
      if (tm != rm || tn != rn || b != rb) { printf("block %u of %d x %d\n", p, s[0], s[1]); return 1; }
    }
  }
  printf("ok\n");
  return 0;
}
"""


def test_block_coords_and_division(tmp_path):
    from paper_2008_13145_amd import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not available")
    src = tmp_path / "geometry.hip"
    src.write_text(SRC)
    exe = tmp_path / "geometry"
    r = subprocess.run([build.HIPCC] + build.CXXFLAGS + ["-I", build.CSRC, str(src), "-o", str(exe)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
