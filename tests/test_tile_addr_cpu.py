"""The kernels' buffer-load addresses of tiled operands (csrc/tile_addr.h), on the host, over every lane: a lane
offset past the buffer's end reads zero and has no uniform offset beside it; any other load lies inside the buffer
with its two offsets added.  The uniform offset alone keeps nothing inside: the bounds check of a buffer load is
only sure to cover the lane offset."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r'''
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include "tile_addr.h"
static void check(const char* what, TileLoad a, unsigned long long bytes, bool there, int x, int y, int z) {
  const bool past = a.lane >= bytes;
  if (past ? (a.uni != 0 || there) : ((unsigned long long)a.lane + a.uni + 16 > bytes || !there)) {
    std::printf("%s: lane %u + uniform %u of %llu bytes, present %d (%d %d %d)\n", what, a.lane, a.uni, bytes, there, x, y, z);
    std::exit(1);
  }
}
int main() {
  // skinny GEMM: N rows of W in blocks of 16, NSUB of them a workgroup; M rows of X padded to 16, MS blocks of them;
  // wt k-tiles, cut into ranges and taken NV steps at a time
  for (int N : {1, 16, 32, 48, 80, 720, 2048})
    for (int nsub : {1, 2, 4})
      for (int wt : {2, 4, 24, 64})
        for (int M : {1, 16, 17, 50, 51, 128, 400})
          for (int nv : {2, 3, 4, 8}) {
            const int blocks = (N + 15) / 16, xt = (M + 15) / 16 * 16, ms = 4;
            const int nt = (blocks + nsub - 1) / nsub, mt = (M + 16 * ms - 1) / (16 * ms);
            for (int tile : {0, nt - 1})
              for (int mtile : {0, mt - 1})
                for (int ke : {(wt + 1) / 2, wt})
                  for (int k = 0; k < ke + nv; ++k)
                    for (int lane = 0; lane < 64; ++lane) {
                      const unsigned lo = (lane & 15) * 64 + (lane >> 4) * 16;
                      const int subs = std::min(blocks - tile * nsub, nsub);
                      for (int s = 0; s < nsub; ++s)
                        check("skinny W", skinny_w_at(lo, s, subs, k, ke, wt), 1024ull * subs * wt, s < subs && k < ke, N, nsub, k);
                      for (int i = 0; i < ms; ++i) {
                        const int row = (mtile * ms + i) * 16;
                        check("skinny X", skinny_x_at(lo, row, xt, k, ke), 64ull * xt * wt, row < xt && k < ke, M, row, k);
                      }
                    }
          }
  // persistent kernel: teams' W of `rows` rows and X of M rows, K cut into chunks of 128 (K <= 1024)
  for (int K : {32, 64, 96, 128, 160, 288, 480, 512, 1024})
    for (int kc = 0; kc < 1024; kc += 128)
      for (int v = 0; v < 4; ++v)
        for (int lane = 0; lane < 64; ++lane) {
          const int r16 = lane & 15;
          const unsigned lo = r16 * 64 + (lane >> 4) * 16;
          const bool k = kc + 32 * v < K;
          for (int rows : {512, 1024})
            for (int row : {0, rows - 16}) {
              check("team W", team_w_at<true>(lo, row, kc, v, K), 2ull * rows * K, k, K, kc, v);
              if (K % 128 == 0 && kc < K) check("team W", team_w_at<false>(lo, row, kc, v, K), 2ull * rows * K, true, K, kc, v);
            }
          for (int M : {1, 16, 17, 50, 64})
            for (int ms = 0; ms < 4; ++ms) {
              const bool in = 16 * ms + r16 < M;
              const TileLoad a = team_x_at<true>(in ? lo : kOob, ms, kc, v, K, M);
              // a subtile's rows share the uniform offset: beside lanes past M it stays the subtile's
              if (in || !k) check("team X", a, 2ull * M * K, in && k, K, kc, v);
              else check("team X past M", {a.lane, 0}, 2ull * M * K, false, K, kc, v);
              if (in && K % 512 == 0 && kc < K) check("team X", team_x_at<false>(lo, ms, kc, v, K, M), 2ull * M * K, true, K, kc, v);
            }
        }
  return 0;
}
'''


def test_tiled_loads_stay_in_their_buffers(tmp_path):
    src = tmp_path / "addr.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "addr")
    subprocess.run(["g++", "-std=c++20", "-O2", "-I", os.path.join(ROOT, "paper_2606_08094_amd", "csrc"), "-o", exe, str(src)],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
