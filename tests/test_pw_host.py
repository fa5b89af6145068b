"""The pointwise products' plan on the host: every pixel that the weight gradient's loads name.

A small C++ program walks the plan of o1d_pw.h as the kernel's threads do (every piece of k, every 16-byte chunk, every
step, and the load past the last step that is issued and never stored) and checks each quad: inside the tensor, whole
quads aligned and within one image, and the pixel that the step's k asks for wherever that k exists.
"""
import os
import subprocess

import pytest

from paper_2309_15812_amd import build

SOURCE = r"""
#include <stdio.h>
#include "o1d_pw.h"
using namespace o1d::pw;

static long long checked = 0, partial = 0;

template <int ES, bool VEC>
static bool walk(int N, int C, int Cout, int H, int W, bool ends = false) {
  const Params P = plan(kWgrad, N, C, Cout, H, W, ES);
  constexpr int BK = kRowBytes / ES, V = 16 / ES;
  if (P.nsplit < 1 || P.per < 1 || (long long)P.steps * BK < P.K || (P.steps - 1ll) * BK >= P.K ||
      (long long)P.per * P.nsplit < P.steps || (P.nsplit - 1ll) * P.per >= P.steps) {
    printf("N=%d H=%d W=%d: %d steps in %d pieces of %d\n", N, H, W, P.steps, P.nsplit, P.per);
    return false;
  }
  for (int split = ends ? P.nsplit - 1 : 0; split < P.nsplit; ++split) {
    const int s0 = split * P.per, s1 = P.steps < s0 + P.per ? P.steps : s0 + P.per;
    if (P.K - s0 * BK < BK) ++partial;  // a piece whose first step is cut
    for (int chunk = 0; chunk < 8; ++chunk) {
      Pixels<ES, VEC> px(P, (unsigned)s0 * BK + chunk * V);
      for (int s = s0; s <= s1; ++s, px.next(P))
        for (int q = 0; q < (int)Pixels<ES, VEC>::NQ; ++q) {
          const long long k = (long long)s * BK + chunk * V + 4 * q;
          const int img = px.img[q], p = px.p[q], run = VEC ? 4 : 1;
          ++checked;
          bool ok = img >= 0 && img < N && p >= 0 && p + run <= P.HW && (!VEC || p % 4 == 0);
          if (k < P.K) ok = ok && img == k / P.HW && p == k % P.HW;
          if (!ok) {
            printf("N=%d C=%d Cout=%d H=%d W=%d bytes=%d vec=%d: piece %d chunk %d step %d quad %d loads pixel %d of "
                   "image %d\n", N, C, Cout, H, W, ES, VEC, split, chunk, s, q, p, img);
            return false;
          }
        }
    }
  }
  return true;
}

int main() {
  const int planes[][2] = {{1, 1}, {1, 4}, {2, 2}, {3, 5}, {4, 4}, {6, 6}, {7, 7}, {7, 8}, {9, 11}, {10, 10}, {14, 14},
                           {18, 18}, {27, 24}, {28, 28}, {45, 37}, {56, 56}};
  const int images[] = {1, 2, 3, 4, 5, 7, 9, 14, 16, 33, 36, 40, 64};
  const int chans[][2] = {{8, 8}, {64, 64}, {100, 36}, {384, 384}, {512, 512}};
  bool ok = true;
  for (auto& hw : planes)
    for (int n : images)
      for (auto& c : chans) {
        const int H = hw[0], W = hw[1];
        ok = ok && walk<4, false>(n, c[0], c[1], H, W) && walk<2, false>(n, c[0], c[1], H, W);
        if (H * W % 4 == 0) ok = ok && walk<4, true>(n, c[0], c[1], H, W) && walk<2, true>(n, c[0], c[1], H, W);
      }
  // images x pixels just below 2^31: the last piece
  ok = ok && walk<4, false>(2, 1, 1, 1, (1 << 30) - 1, true) && walk<2, false>(2, 1, 1, 1, (1 << 30) - 1, true) &&
       walk<4, false>(1, 1, 8, 1, 2147483647, true) && walk<4, true>(1, 1, 8, 1, 2147483644, true) &&
       walk<2, true>(1, 1, 8, 1, 2147483644, true);
  // and the grid over their columns
  for (int kind : {kFwd, kDgrad}) {
    const Params P = plan(kind, 1, 1, 8, 1, 2147483647, 4);
    const long long x = grid_x(P), y = grid_y(P);
    if (P.nblocks != 1 << 24 || x * y < P.nblocks || x * kThreads >= 1ll << 32 || y > 65535 || x * y >= 1ll << 31) {
      printf("grid %lld x %lld for %d workgroups\n", x, y, P.nblocks);
      ok = false;
    }
  }
  printf("%s: %lld quads, %lld pieces that start on a cut step\n", ok ? "ok" : "bad", checked, partial);
  return ok && partial > 0 ? 0 : 1;
}
"""


@pytest.fixture(scope="module")
def compile_run(tmp_path_factory):
    def go(source):
        d = tmp_path_factory.mktemp("pw")
        src, exe = d / "t.cpp", d / "t"
        src.write_text(source)
        rocm = os.path.dirname(os.path.dirname(os.path.realpath(build.HIPCC)))
        subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", build.CSRC,
                        "-I", os.path.join(rocm, "include"), str(src), "-o", str(exe)], check=True)
        return subprocess.run([str(exe)], capture_output=True, text=True)
    return go


def test_weight_gradient_loads_stay_in_the_tensor(compile_run):
    r = compile_run(SOURCE)
    assert r.returncode == 0, r.stdout


SUMS = r"""
#include <stdio.h>
#include "o1d_pw.h"
using namespace o1d::pw;
// float32 pieces of k: length plus number (the square of a sum's error grows with them) no more than with whole images,
// except where a piece is a single step already
int main() {
  const int planes[][2] = {{3, 3}, {7, 7}, {7, 9}, {8, 8}, {9, 21}, {12, 12}, {14, 14}, {28, 28}, {56, 56}};
  const int chans[][2] = {{8, 8}, {64, 64}, {384, 384}, {512, 512}, {13, 253}};
  for (auto& hw : planes)
    for (int n : {1, 2, 5, 8, 16, 33, 64, 3000})
      for (auto& c : chans) {
        const Params P = plan(kWgrad, n, c[0], c[1], hw[0], hw[1], 4);
        const int want = cdiv(1024, cdiv(c[0], kTile) * cdiv(c[1], kTile)), groups = n < want ? n : want;
        const int images = cdiv(n, groups);
        if (P.per > 1 && 32 * P.per + P.nsplit > images * hw[0] * hw[1] + cdiv(n, images)) {
          printf("N=%d %dx%d C=%d: %d pieces of %d steps\n", n, hw[0], hw[1], c[0], P.nsplit, P.per);
          return 1;
        }
      }
  return 0;
}
"""


def test_float32_pieces_are_no_longer_than_whole_images(compile_run):
    r = compile_run(SUMS)
    assert r.returncode == 0, r.stdout
