"""The launch geometry of the token layout's kernels (host code of cg_device.h) against the limit of
a HIP launch, fewer than 2^32 threads: a shape that one wave per 64 tokens and per 64 channels can
launch is launchable."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SRC = r"""
#include <cstdio>
#include "cg_device.h"
int main() {
  const size_t lds[4] = {10000, 15000, 25000, 45000};
  const int tokens[] = {1, 31, 32, 64, 65, 257, 320, 321, 513, 1536};
  const int channels[] = {1, 8, 63, 64, 65, 128, 136, 1024};
  const int groups[] = {1, 7, 10, 100};
  int shapes = 0, bad = 0;
  for (int n : tokens)
    for (int C : channels)
      for (int G : groups)
        for (int lg = 10; lg <= 26; ++lg)
          for (int odd = 0; odd <= 1; ++odd) {
            KParams P = {};
            P.B = 1; P.L = 1; P.C = C; P.G = G; P.CL = n; P.nblk = (C + 63) / 64;
            P.NC = (1 << (lg - 1)) + odd;              // chunks: 2 NC rows
            if ((long long)P.NC * n > 0x7fffffffll) continue;
            P.T = P.NC * n;
            const long long rows = 2ll * P.NC, nbj = (n + 63) / 64;
            const TokGrid t = cg_tok_grid(P, (int)nbj, lds);
            const bool one = rows * nbj * 64 <= 0xFFFFFFFFll;       // a wave per 64 tokens
            if (one && t.grid * t.w * 64 > 0xFFFFFFFFll) { ++bad; printf("tokens n=%d C=%d rows=%lld w=%d\n", n, C, rows, t.w); }
            for (int vec = 0; vec <= (C % 8 == 0); ++vec) {
              const TokRowGrid g = cg_tok_row_grid(P, vec);
              const bool row = rows * P.nblk * 64 <= 0xFFFFFFFFll;  // a wave per 64 channels
              if (g.threads < 64 || g.threads > 512 || g.threads % 64) { ++bad; printf("threads %d\n", g.threads); }
              if (row && g.grid * g.threads > 0xFFFFFFFFll) { ++bad; printf("rows n=%d C=%d G=%d rows=%lld threads=%d\n", n, C, G, rows, g.threads); }
            }
            ++shapes;
          }
  printf("%d shapes, %d bad\n", shapes, bad);
  return bad != 0 || shapes < 1000;
}
"""


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which(HIPCC)), reason="no hipcc")
def test_token_layout_launches_stay_below_2_32_threads(tmp_path):
    src = tmp_path / "geom.hip"
    src.write_text(SRC)
    exe = tmp_path / "geom"
    subprocess.run([HIPCC, "--offload-host-only", "-std=c++17", "-O1", "-w", "-I",
                    os.path.join(ROOT, "paper_2310_07240_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
