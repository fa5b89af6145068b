// Device code of the pointwise convolution's matrix products (included by
// o1d_pw_f32.hip and o1d_pw_bf16.hip); the host plan is in o1d_pw.h.
//
// A workgroup computes a 128 x 128 tile of the output with four waves, each
// 32 rows x 128 columns (four 32 x 32 matrix-core accumulators).  Per step
// 128 bytes of k (32 float32, 64 bfloat16) of 128 rows of A and 128 columns
// of B are staged in LDS as rows of k, 144 bytes apart, so that every LDS
// access is a 16-byte one and eight lanes' accesses (36 words apart, or one
// row) cover all 32 banks.  The next step's loads are in flight during a
// step's products.  One buffer of 36 KB and three workgroups per CU: two
// buffers with one barrier per step leave two per CU, which was slower (fwd
// at the shape below 943 against 909 us).
// float32 storage multiplies on v_mfma_f32_32x32x2_f32 (float32 products),
// bfloat16 storage on v_mfma_f32_32x32x16_bf16; both accumulate in float32.
//
// Operands whose memory runs along rows instead of k (B of the forward and
// the input gradient, Wp of the input gradient) are loaded as blocks of four
// rows x 16 bytes of k per thread and transposed in registers; thread
// (g, kg) holds rows 4 g .. 4 g + 3, and row 4 g + e lies at LDS row
// g + 32 e.  A wave's four accumulators then hold four consecutive columns
// per lane, which leave as one vector store.  (Columns that take element
// accesses, odd planes say, are g + 32 e instead: 10 x 16 -> 104 x 189 x 113,
// bfloat16, block forward 88 -> 84 us.)
//
// The k of one 16-byte LDS chunk need not be consecutive matrix-core steps:
// half-wave h takes chunks 2 j + h of A and of B alike, element s of the two
// chunks forming float32 step (j, s).
//
// What bounds it: the matrix cores in float32 (64 cycles per instruction).
// 64 x 512 -> 512 x 56 x 56 (105 GFLOP per product), float32: forward 1158 ->
// 920 us (114 TFLOP/s), the backward's two products 2280 -> 1730 us (122; the
// library's largest float32 product reaches 153); bfloat16, 64 x 384 -> 384 x
// 14 x 14: 42 -> 16 us per product.  Before, loads behind per-run range tests
// were waited for one by one, LDS took 4-byte accesses, and every image ended
// in a partly used tile.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

#include "o1d_device.h"
#include "o1d_pw.h"

namespace o1d {
namespace pw {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <typename T, bool VEC>
using Pix = Pixels<(int)sizeof(T), VEC>;

constexpr int kPitch = 144;                   // bytes between LDS rows
constexpr int kBuf = 2 * kTile * kPitch;      // one buffer: A rows, then B rows

template <typename T>
struct Fmt {
  static constexpr int V = 16 / (int)sizeof(T);            // k per chunk
  static constexpr int BK = kRowBytes / (int)sizeof(T);    // k per step
  static constexpr int QW = (int)sizeof(T);                // 32-bit words of four elements
};

// Four consecutive elements as packed words: one vector access, or (runs that
// are not whole or not aligned) the elements at p + off(e).  Loads are never
// conditional: what a share has past the operand's end is loaded from a
// clamped address, and only the k past the end are cleared (`clear`), in the
// last step: a register that a load may or may not write would make the
// compiler wait for every load before the next.
template <typename T, bool VEC, class F>
__device__ __forceinline__ void load_quad(const T* p, F&& off, uint32_t* w) {
  if constexpr (VEC) {
    __builtin_memcpy(w, __builtin_assume_aligned(p + off(0), 4 * sizeof(T)), 4 * sizeof(T));
  } else {
    T t[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] = p[off(e)];
    __builtin_memcpy(w, t, sizeof(t));
  }
}

// A thread's share of one operand's tile: 16 words.
// Rows of k (kc): chunks kq = t % 8 of rows t / 8 + 32 i.
// Runs along rows (rc): rows 4 g .. 4 g + 3 (g = t % 32), chunk kg = t / 32.
struct Share {
  uint32_t v[16];
};

// Clears the elements whose k is past the operand's last (`left` of the
// step's k exist, the share holds those of chunk `chunk`): chunks of k (kc) or
// rows of k (rc).
template <typename T, bool RC>
__device__ __forceinline__ void clear_past(Share& s, int left, int chunk) {
  constexpr int V = Fmt<T>::V, QW = Fmt<T>::QW;
  const int k = chunk * V;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    if constexpr (RC) {
      if (k + i / QW >= left) s.v[i] = 0u;
    } else if constexpr (sizeof(T) == 4) {
      if (k + i % 4 >= left) s.v[i] = 0u;
    } else {
      const int e = k + 2 * (i % 4);
      s.v[i] = e + 1 < left ? s.v[i] : (e < left ? s.v[i] & 0xffffu : 0u);
    }
  }
}

__device__ __forceinline__ void put16(char* lds, const uint32_t* w) {
  u32x4 x;
  x[0] = w[0]; x[1] = w[1]; x[2] = w[2]; x[3] = w[3];
  *reinterpret_cast<u32x4*>(lds) = x;
}

// SPREAD: row m lies at LDS row 32 (m % 4) + m / 4, as the transposed rows do,
// so that each wave has a quarter of the rows of an operand of few.
template <bool SPREAD = false>
__device__ __forceinline__ void store_kc(const Share& s, char* lds) {
  const int t = threadIdx.x;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = t / 8 + 32 * i;
    put16(lds + (SPREAD ? 32 * (row % 4) + row / 4 : row) * kPitch + (t % 8) * 16, &s.v[4 * i]);
  }
}

// rc shares hold V rows of k x E elements, in places of four; the transpose
// picks element e of every k.  Element e is the operand's e0 + e.
template <typename T, int E = 4>
__device__ __forceinline__ void store_rc(const Share& s, char* lds, int chunk, int e0) {
  const int g = threadIdx.x % 32;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (sizeof(T) == 4) {
        w[i] = s.v[4 * i + e];
      } else {
        // k 2 i and 2 i + 1: halves e of the quads s.v[4 i ..] and s.v[4 i + 2 ..]
        const uint32_t a = s.v[4 * i + (e >> 1)], b = s.v[4 * i + 2 + (e >> 1)];
        w[i] = (e & 1) ? (a >> 16) | (b & 0xffff0000u) : (a & 0xffffu) | (b << 16);
      }
    }
    put16(lds + (g + 32 * (e0 + e)) * kPitch + chunk * 16, w);
  }
}

// Element accesses are many (32 loads per thread and operand in bfloat16), so
// a wave whose rows or k all lie past the operand's end leaves them out.
__device__ __forceinline__ int first_of_wave(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Rows of Wp (contiguous along k): row r, k from k0 of this step.
template <typename T, bool VEC>
__device__ __forceinline__ void load_w_kc(const Params& P, const T* __restrict__ A, int row0, int k0, Share& s) {
  constexpr int V = Fmt<T>::V, QW = Fmt<T>::QW;
  const int t = threadIdx.x, k = k0 + (t % 8) * V;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (!VEC && first_of_wave(row0 + t / 8 + 32 * i) >= P.M) break;  // rows that are not stored
    const long long r = (long long)min(row0 + t / 8 + 32 * i, P.M - 1) * P.K;
#pragma unroll
    for (int q = 0; q < V / 4; ++q)
      load_quad<T, VEC>(A, [&](int e) { return r + min(k + 4 * q + e, VEC ? P.K - 4 : P.K - 1); }, &s.v[4 * i + QW * q]);
  }
}

// Columns of Wp (the input gradient's A: element (m, k) at k M + m).
template <typename T, bool VEC>
__device__ __forceinline__ void load_w_rc(const Params& P, const T* __restrict__ A, int row0, int k0, Share& s) {
  constexpr int V = Fmt<T>::V, QW = Fmt<T>::QW;
  const int r = row0 + 4 * (threadIdx.x % 32), k = k0 + (threadIdx.x / 32) * V;
  if (!VEC && first_of_wave(k) >= P.K) return;  // cleared before they are stored
#pragma unroll
  for (int i = 0; i < V; ++i) {
    const long long row = (long long)min(k + i, P.K - 1) * P.M;
    load_quad<T, VEC>(A, [&](int e) { return row + min(r + e, VEC ? P.M - 4 : P.M - 1); }, &s.v[QW * i]);
  }
}

// B of the forward and the input gradient, and their outputs: column (image,
// pixel), rows HW apart.  Thread g's four columns of a tile (n0 on), which lie
// at LDS rows g + 32 e: 4 g + e where they are one access (VEC), else g + 32 e
// from e0 on, so that an element access covers consecutive pixels over the
// lanes.  off[e]: element offset of column e (the last column's where there is
// none; off[0] alone where VEC).
template <bool VEC>
struct Cols {
  long long off[4];
  bool in[4];
  __device__ __forceinline__ Cols(const Params& P, long long n0, int g0, int ch, int e0) {
#pragma unroll
    for (int e = 0; e < (VEC ? 1 : 4); ++e) {
      const long long col = n0 + (VEC ? 4 * g0 : g0 + 32 * (e0 + e));
      in[e] = col < P.N;
      const int g = (int)(in[e] ? col : P.N - (VEC ? 4 : 1));  // (images x pixels stay below 2^31)
      const int img = g / P.HW;
      off[e] = (long long)img * ch * P.HW + (g - img * P.HW);
    }
  }
};

// Rows k on of the first E columns.
template <typename T, bool VEC, int E = 4>
__device__ __forceinline__ void load_cols(const Params& P, const T* __restrict__ B, const Cols<VEC>& c, int k,
                                          Share& s) {
  constexpr int V = Fmt<T>::V, QW = Fmt<T>::QW;
  if (!VEC && first_of_wave(k) >= P.K) return;  // cleared before they are stored
#pragma unroll
  for (int i = 0; i < V; ++i) {
    const long long row = (long long)min(k + i, P.K - 1) * P.HW;
    if constexpr (E == 4) {
      load_quad<T, VEC>(B, [&](int e) { return row + c.off[e]; }, &s.v[QW * i]);
    } else {
      T t[4] = {};
#pragma unroll
      for (int e = 0; e < E; ++e) t[e] = B[row + c.off[e]];
      __builtin_memcpy(&s.v[QW * i], t, sizeof(t));
    }
  }
}

// The weight gradient's operands: rows are channels, k = (image, pixel).
template <typename T, bool VEC>
__device__ __forceinline__ void load_pix(const Params& P, const T* __restrict__ X, int rows, int row0,
                                         const Pix<T, VEC>& px, Share& s) {
  constexpr int QW = Fmt<T>::QW;
  const int t = threadIdx.x;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (!VEC && first_of_wave(row0 + t / 8 + 32 * i) >= rows) break;  // rows that are not stored
    const int r = min(row0 + t / 8 + 32 * i, rows - 1);
#pragma unroll
    for (int q = 0; q < (int)Pix<T, VEC>::NQ; ++q) {
      load_quad<T, VEC>(X, [&](int e) {
        int img = px.img[q], p = px.p[q];
        if (!VEC && px.k + 4 * q + e < (unsigned)P.K) {  // elements of a run may lie in the next images
          p += e;
          while (p >= P.HW) {
            p -= P.HW;
            ++img;
          }
        }
        return ((long long)img * rows + r) * P.HW + p;
      }, &s.v[4 * i + QW * q]);
    }
  }
}

// One step's products of the wave's 32 x 128 block from a staged buffer.  A
// chunk's reads are issued before the products of the chunk before it.
struct Frag {
  u32x4 a, b[4];
  __device__ __forceinline__ void read(const char* a0, const char* b0, int j) {
    a = *reinterpret_cast<const u32x4*>(a0 + 32 * j);
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) b[nb] = *reinterpret_cast<const u32x4*>(b0 + nb * 32 * kPitch + 32 * j);
  }
};

template <typename T>
__device__ __forceinline__ void products(const Frag& f, f32x16 (&acc)[4]) {
  if constexpr (sizeof(T) == 4) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int nb = 0; nb < 4; ++nb)
        acc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(f.a[s]), __uint_as_float(f.b[nb][s]), acc[nb], 0,
                                                       0, 0);
  } else {
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
      acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f.a),
                                                        __builtin_bit_cast(bf16x8, f.b[nb]), acc[nb], 0, 0, 0);
  }
}

// `chunks`: the step's chunks of k that hold any (all of them where SHORT is not set).
template <typename T, bool SHORT>
__device__ __forceinline__ void multiply(const char* buf, int chunks, f32x16 (&acc)[4]) {
  const int l = threadIdx.x & 63, r = l & 31, h = l >> 5, w = threadIdx.x >> 6;
  const char* a0 = buf + (32 * w + r) * kPitch + 16 * h;
  const char* b0 = buf + (kTile + r) * kPitch + 16 * h;
  constexpr int NJ = kRowBytes / 32;
  Frag f[2];
  f[0].read(a0, b0, 0);
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    if (SHORT && j > 0 && 2 * j >= chunks) break;
    if (j + 1 < NJ) f[(j + 1) & 1].read(a0, b0, j + 1);
    products<T>(f[j & 1], acc);
  }
}

// VA, VB: A's and B's (and the output's) runs of four elements are whole and aligned.
template <typename T, int KIND, bool VA, bool VB>
__global__ __launch_bounds__(kThreads, VB || sizeof(T) == 2 ? 3 : 2) void pw_gemm(Params P, const T* __restrict__ A,
                                                                                  const T* __restrict__ B,
                                                                                  void* __restrict__ out) {
  extern __shared__ __align__(16) char lds[];
  constexpr int BK = Fmt<T>::BK;
  // Rows of the output over the waves.  (The forward's vector stores keep 32
  // rows per wave; its element stores, four times as many, are shared out.)
  constexpr bool kSpread = KIND == kDgrad || (KIND == kFwd && !VB);
  // tiles along M are neighbours on one XCD: they share B's columns in its L2
  // (past the last one: that tile again, not stored; a branch here instead of
  // at the end puts the arguments' loads in series, 0.4% of the product)
  const int at = (int)(blockIdx.y * kGridRow + blockIdx.x), b = min(at, P.nblocks - 1);
  const int id = P.xcd_per ? (b % 8) * P.xcd_per + b / 8 : b;
  const int mt = id % P.tm, rest = id / P.tm;
  const int split = rest % P.nsplit, nt = rest / P.nsplit;
  const int m0 = mt * kTile;
  const long long n0 = (long long)nt * kTile;
  const int s0 = split * P.per, s1 = min(P.steps, s0 + P.per);
  Pix<T, VA> px(P, KIND == kWgrad ? (unsigned)s0 * BK + (threadIdx.x % 8) * Fmt<T>::V : 0u);
  // B's element loads, 32 per thread in bfloat16, are shared out over all waves
  // where few channels fill only the first chunks: E columns from e0 on of
  // chunk `chunk` (58 x 10 -> 10 x 59 x 59, bfloat16: block forward 41 -> 29 us)
  const int kg = threadIdx.x / 32;
  const int nc = !VB && KIND != kWgrad ? chunks_of(P.K, (int)sizeof(T)) : 8;
  const int chunk = VB ? kg : kg & (nc - 1), e0 = VB ? 0 : first_of_wave(kg / nc) * (nc / 2);
  const Cols<VB> cols(P, KIND == kWgrad ? 0 : n0, threadIdx.x % 32, P.rowsB, e0);
  auto with_cols = [&](auto&& f) __attribute__((always_inline)) {
    if constexpr (VB) {
      f(std::integral_constant<int, 4>());
    } else {
      if (nc == 8)
        f(std::integral_constant<int, 4>());
      else if (nc == 4)
        f(std::integral_constant<int, 2>());
      else
        f(std::integral_constant<int, 1>());
    }
  };
  Share sa, sb;
  auto load = [&](int s) __attribute__((always_inline)) {
    if constexpr (KIND == kWgrad) {
      load_pix<T, VA>(P, A, P.rowsA, m0, px, sa);
      load_pix<T, VB>(P, B, P.rowsB, (int)n0, px, sb);
      px.next(P);
    } else {
      if constexpr (KIND == kFwd)
        load_w_kc<T, VA>(P, A, m0, s * BK, sa);
      else
        load_w_rc<T, VA>(P, A, m0, s * BK, sa);
      with_cols([&](auto e) __attribute__((always_inline)) {
        load_cols<T, VB, decltype(e)::value>(P, B, cols, s * BK + chunk * Fmt<T>::V, sb);
      });
    }
  };
  auto store = [&](char* buf, int s) __attribute__((always_inline)) {
    const int left = P.K - s * BK;
    if (left < BK) {
      clear_past<T, KIND == kDgrad>(sa, left, KIND == kDgrad ? kg : threadIdx.x % 8);
      clear_past<T, KIND != kWgrad>(sb, left, KIND != kWgrad ? chunk : threadIdx.x % 8);
    }
    if constexpr (KIND == kDgrad)
      store_rc<T>(sa, buf, kg, 0);
    else
      store_kc<kSpread>(sa, buf);
    if constexpr (KIND == kWgrad)
      store_kc(sb, buf + kTile * kPitch);
    else
      with_cols([&](auto e) __attribute__((always_inline)) {
        store_rc<T, decltype(e)::value>(sb, buf + kTile * kPitch, chunk, e0);
      });
  };
  f32x16 acc[4];
#pragma unroll
  for (int nb = 0; nb < 4; ++nb)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[nb][e] = 0.f;
  load(s0);
  for (int s = s0; s < s1; ++s) {
    __syncthreads();  // the previous step's reads are done
    store(lds, s);
    // in flight during the products (vector loads past the last step load
    // something in range that is never stored; element loads are left out)
    if (VB || s + 1 < s1) load(min(s + 1, s1 - 1));
    __syncthreads();
    multiply<T, !VB && KIND != kWgrad>(lds, nc, acc);
  }
  if (at >= P.nblocks) return;
  const int l = threadIdx.x & 63, r = l & 31, w = threadIdx.x >> 6;
  if constexpr (KIND == kWgrad) {
    float* o = static_cast<float*>(out) + (long long)split * P.M * P.N;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int m = m0 + 32 * w + 8 * (e >> 2) + 4 * (l >> 5) + (e & 3);
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) {
        const int n = (int)n0 + 32 * nb + r;
        if (m < P.M && n < P.N) o[(long long)m * P.N + n] = acc[nb][e];
      }
    }
  } else {
    const Cols<VB> oc(P, n0, r, P.M, 0);
    T* o = static_cast<T*>(out);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int row = 8 * (e >> 2) + 4 * (l >> 5) + (e & 3);
      const int m = m0 + (kSpread ? 4 * row + w : 32 * w + row);
      if (m >= P.M) continue;
      T t[4];
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) t[nb] = from_f32<T>(acc[nb][e]);
      const long long ro = (long long)m * P.HW;
      if constexpr (VB) {
        if (oc.in[0]) __builtin_memcpy(__builtin_assume_aligned(o + oc.off[0] + ro, 4 * sizeof(T)), t, sizeof(t));
      } else {
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
          if (oc.in[nb]) o[oc.off[nb] + ro] = t[nb];
      }
    }
  }
}

template <typename T, int KIND, bool VA, bool VB>
hipError_t launch_kind(const Params& p, const void* A, const void* B, void* out, hipStream_t stream) {
  static std::atomic<int> allowed{0};
  if (!allowed.load(std::memory_order_acquire)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(pw_gemm<T, KIND, VA, VB>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, kBuf);
    if (e != hipSuccess) return e;
    allowed.store(1, std::memory_order_release);
  }
  hipLaunchKernelGGL((pw_gemm<T, KIND, VA, VB>), dim3(grid_x(p), grid_y(p)), dim3(kThreads), kBuf, stream, p,
                     static_cast<const T*>(A), static_cast<const T*>(B), out);
  return hipGetLastError();
}

// Runs of four elements: pixels come in fours and the tensors are aligned to
// a run; Wp's rows (forward: K elements, input gradient: M) likewise.
template <typename T>
hipError_t gemm_t(int kind, const Params& p, const void* A, const void* B, void* out, hipStream_t stream) {
  auto quads = [](const void* t) { return (uintptr_t)t % (4 * sizeof(T)) == 0; };
  if (kind == kWgrad)
    return p.HW % 4 == 0 && quads(A) && quads(B) ? launch_kind<T, kWgrad, true, true>(p, A, B, out, stream)
                                                 : launch_kind<T, kWgrad, false, false>(p, A, B, out, stream);
  const bool vb = p.HW % 4 == 0 && quads(B) && quads(out), va = (kind == kFwd ? p.K : p.M) % 4 == 0 && quads(A);
  if (kind == kFwd) {
    if (va) return vb ? launch_kind<T, kFwd, true, true>(p, A, B, out, stream)
                      : launch_kind<T, kFwd, true, false>(p, A, B, out, stream);
    return vb ? launch_kind<T, kFwd, false, true>(p, A, B, out, stream)
              : launch_kind<T, kFwd, false, false>(p, A, B, out, stream);
  }
  if (va) return vb ? launch_kind<T, kDgrad, true, true>(p, A, B, out, stream)
                    : launch_kind<T, kDgrad, true, false>(p, A, B, out, stream);
  return vb ? launch_kind<T, kDgrad, false, true>(p, A, B, out, stream)
            : launch_kind<T, kDgrad, false, false>(p, A, B, out, stream);
}

}  // namespace
}  // namespace pw
}  // namespace o1d
