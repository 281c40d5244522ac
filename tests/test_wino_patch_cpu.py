"""The 4x4 input patch of a Winograd tile, run on the host: every position it
loads lies inside the image, also where the image has no rows or no columns and
the patch lies in the padding alone, and its values are those of the
zero-padded image."""
import os
import subprocess

import pytest

SRC = r"""
#include <cstdio>
#include <cstdint>
#include "wino_patch.hpp"
template <typename I>
static int check() {
  for (I H = 0; H <= 6; ++H)
    for (I W = 0; W <= 6; ++W)
      for (I pad = 0; pad <= 4; ++pad)
        for (I y0 = -pad; y0 < H + pad; ++y0)
          for (I x0 = -pad; x0 < W + pad; ++x0) {
            int outside = 0, loads = 0;
            float v[4][4];
            kt::wino_patch(H, W, y0, x0, 0.f, [&](I y, I x) {
              ++loads;
              if (y < 0 || y >= H || x < 0 || x >= W) { ++outside; return -1.f; }
              return (float)(1 + y * W + x);
            }, v);
            if (outside) { printf("%d of %d loads outside %d x %d\n", outside, loads, (int)H, (int)W); return 1; }
            for (int u = 0; u < 4; ++u)
              for (int w = 0; w < 4; ++w) {
                const I y = y0 + u, x = x0 + w;
                const bool in = y >= 0 && y < H && x >= 0 && x < W;
                if (v[u][w] != (in ? (float)(1 + y * W + x) : 0.f)) { printf("value\n"); return 1; }
              }
          }
  return 0;
}
int main() {
  if (check<int32_t>() || check<int64_t>()) return 1;
  printf("ok\n");
  return 0;
}
"""


def test_patch_stays_inside_the_image(tmp_path):
    from paper_2008_13145_amd import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not available")
    src = tmp_path / "patch.hip"
    src.write_text(SRC)
    exe = tmp_path / "patch"
    r = subprocess.run([build.HIPCC] + build.CXXFLAGS + ["-I", build.CSRC, str(src), "-o", str(exe)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
