// Host-side plan of the pointwise (1 x 1) convolution of the oriented 1D
// depthwise separable block (Sec. 3.2, "Computational cost analysis", and
// Table 1's "Oriented 1D DSC"): dense contractions over channels or pixels,
// run as matrix products C[m][n] = sum_k A[m][k] B[k][n] on the matrix cores.
//
//   kFwd    Y  = Wp   Z    M = C',  n = (image, pixel),  K = C
//   kDgrad  dZ = Wp^T dY   M = C,   n = (image, pixel),  K = C'
//   kWgrad  dWp = dY Z^T   M = C',  N = C,               k = (image, pixel)
//
// (image, pixel) is one index over all images, so that planes that are no
// multiple of a tile leave no partly used tile per image.  The weight
// gradient's k range is cut into nsplit pieces whose float32 partial results
// are added in a fixed order.
#pragma once

#include <stddef.h>

#include "o1d_launch.h"
#include "o1d_plan.h"

namespace o1d {
namespace pw {

enum Kind { kFwd = 0, kDgrad = 1, kWgrad = 2 };

constexpr int kThreads = 256;  // four waves, each 32 rows x all 128 columns of the tile
constexpr int kTile = 128;     // tile rows and columns
constexpr int kRowBytes = 128; // k per step: 32 float32 or 64 bfloat16

struct Params {
  int M, K;          // output rows; contraction length (weight gradient: images x pixels)
  long long N;       // output columns (forward, input gradient: images x pixels)
  int HW;            // pixels per image
  int rowsA, rowsB;  // weight gradient: channels of dY and Z; else rowsB: channels of B, M: channels of the output
  int tm;            // tiles along M (the fastest index: they share B's columns)
  int steps, per;    // k steps in all and per workgroup
  int nsplit;        // weight gradient: pieces of k
  int nblocks, xcd_per;
};

// (64-bit sums: images x pixels may be anything below 2^31)
inline int cdiv(long long a, int b) { return (int)((a + b - 1) / b); }

// The product for N images of C -> Cout channels; esize: bytes per element.
inline Params plan(int kind, int N, int C, int Cout, int H, int W, int esize) {
  Params p{};
  p.HW = H * W;
  const int bk = kRowBytes / esize;
  const long long pix = (long long)N * p.HW;
  if (kind == kWgrad) {
    p.M = Cout;
    p.N = C;
    p.rowsA = Cout;
    p.rowsB = C;
    p.K = (int)pix;
  } else {
    p.M = kind == kFwd ? Cout : C;
    p.K = kind == kFwd ? C : Cout;
    p.rowsB = p.K;
    p.N = pix;
  }
  p.tm = cdiv(p.M, kTile);
  const int tn = cdiv(p.N, kTile);
  p.steps = cdiv(p.K, bk);
  p.per = p.steps;
  if (kind == kWgrad) {
    // pieces of k: about 1024 workgroups in float32, 512 in bfloat16 (half
    // the partial results to write and add; their rounding is far below the
    // bfloat16 result's); at least four steps each, or in bfloat16 one where
    // odd planes take element loads, whose steps are long (5 x 103 -> 17 x 11 x
    // 11: block backward 55 -> 30 us)
    const int want = cdiv(esize == 4 ? 1024 : 512, p.tm * tn);
    const int most = esize == 2 && p.HW % 4 ? p.steps : p.steps / 4, pieces = want < most ? want : most;
    p.per = cdiv(p.steps, pieces > 1 ? pieces : 1);
    if (esize == 4) {
      // The square of a float32 sum's error grows with the piece's length
      // plus the number of pieces.  Pieces are cut until that is no more than
      // with whole images (up to `want` of them): 16 x 512 -> 512 x 7 x 7 has
      // 1.5e-7 against float64 with pieces of an image, 2.3e-7 with four steps.
      const int whole = cdiv(N, N < want ? N : want);
      const long long limit = (long long)p.HW * whole + cdiv(N, whole);
      while (p.per > 1 && (long long)bk * p.per + cdiv(p.steps, p.per) > limit) --p.per;
    }
  }
  p.nsplit = cdiv(p.steps, p.per);
  p.nblocks = p.tm * tn * p.nsplit;
  p.xcd_per = p.nblocks % 8 == 0 ? p.nblocks / 8 : 0;
  return p;
}

// 16-byte chunks of k that one step holds at least (2, 4 or all 8): with fewer
// the products stop there, and where B takes element loads a chunk's four
// columns per thread are shared out over the threads of the absent chunks.
__host__ __device__ inline int chunks_of(int K, int esize) {
  const int v = 16 / esize;
  return K <= 2 * v ? 2 : (K <= 4 * v ? 4 : 8);
}

// Launch grid: rows of at most 2^22 workgroups, as the workitems of one
// dimension stay below 2^32; the last row's excess stores nothing.
constexpr int kGridRow = 1 << 22;
inline unsigned grid_x(const Params& p) { return (unsigned)(p.nblocks < kGridRow ? p.nblocks : kGridRow); }
inline unsigned grid_y(const Params& p) { return (unsigned)cdiv(p.nblocks, kGridRow); }

// The weight gradient's k = (image, pixel): a thread's 16-byte chunk of k
// (ES: bytes per element) as quads of four, the same chunk of every step from
// k0 on.  Quad q is loaded from pixel p[q] of image img[q]; a quad past the
// last k repeats the last one that is whole (VEC: a quad is one access of four
// pixels of one image, so H W and every k0 are multiples of four) or the last
// pixel (single elements).  (Unsigned: k may pass 2^31 by a step.)
template <int ES, bool VEC>
struct Pixels {
  static constexpr unsigned NQ = 4 / ES;
  static constexpr unsigned BK = kRowBytes / ES;
  unsigned k;
  int img[NQ], p[NQ];
  __host__ __device__ __forceinline__ Pixels(const Params& P, unsigned k0) {
    k = k0;
#pragma unroll
    for (unsigned q = 0; q < NQ; ++q) {
      const unsigned last = (unsigned)P.K - (VEC ? 4 : 1);
      const int at = (int)(k + 4 * q < last ? k + 4 * q : last);
      img[q] = at / P.HW;
      p[q] = at - img[q] * P.HW;
    }
  }
  __host__ __device__ __forceinline__ void next(const Params& P) {
    k += BK;
#pragma unroll
    for (unsigned q = 0; q < NQ; ++q) {
      if (k + 4 * q < (unsigned)P.K) {
        p[q] += (int)BK;
        while (p[q] >= P.HW) {
          p[q] -= P.HW;
          ++img[q];
        }
      }
    }
  }
};

}  // namespace pw

// One translation unit per storage type; see o1d_pw_kernels.h.  `out` is
// the output tensor, or for kWgrad the float32 partials nsplit x M x N, which
// launch_partial_sum then adds into the output.
#define O1D_PW_DECL(T)                                                                                       \
  hipError_t launch_pw_gemm_##T(int kind, const pw::Params& p, const void* A, const void* B, void* out,      \
                                hipStream_t stream);
O1D_PW_DECL(f32)
O1D_PW_DECL(bf16)
#undef O1D_PW_DECL

inline hipError_t launch_pw_gemm(Dtype dt, int kind, const pw::Params& p, const void* A, const void* B, void* out,
                                 hipStream_t stream) {
  return dt == Dtype::F32 ? launch_pw_gemm_f32(kind, p, A, B, out, stream)
                          : launch_pw_gemm_bf16(kind, p, A, B, out, stream);
}

}  // namespace o1d
