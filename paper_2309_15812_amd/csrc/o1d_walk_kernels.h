// Device code of the walk kernels (included by the translation units
// o1d_walk_{f32,bf16}_{nchw,nhwc}.hip); the host plan is in o1d_walk.h.
//
// The operation (Definition 1, Eq. 1-2) is a list of cells per channel: a
// cell is an integer offset (a, b) (Eq. 2's rounded-down offsets of a tap, or
// one corner of the bilinear interpolation of the section "Discretization
// and Interpolation") with the weight w_k coef, equal offsets merged:
// y[p,q] = sum over cells of weight x[str p + a, str q + b].
//
// Phases.  With a = str a' + pi and b = str b' + pj (0 <= pi, pj < str) the
// cells of phase (pi, pj) are a stride-1 list (a', b') on the source's
// sub-lattice (str i + pi, str j + pj); the input gradient's output phase
// (pi, pj) gathers dy with the cells (-a', -b') of the same phase.
//
// Program (one per channel, in LDS, built once per workgroup by one wave
// with a lane per row of the line in the staging frame, whose rows run along
// the line's longer extent): per phase the row's cells form up to four
// chains (the row's first column, the next one, ...).  Walking a chain, a
// cell that is its predecessor moved by u = (1, s) continues the window of
// the strip walk; any other cell starts a run.  Cells are kept in chunks of
// 32 whose first cell starts a run, so a walk of any length is a loop over
// one unrolled chunk.
//
// A team's lanes compute blocks of NC adjacent strips of R outputs (the
// strip kernels' shapes); a workgroup stages its teams' tiles together, a
// row of the plane at a time, with buffer accesses whose range check gives
// the zeros outside the plane.
//
// Measured against the table kernels (kernel trace, us): NHWC 64 x 96 x 56 x
// 56, K = 31, float32: forward 259 -> 128, weight gradient 277 -> 134; NHWC 64 x
// 384 x 14 x 14, bfloat16: 86 -> 42, 171 -> 43; bilinear at the first shape: 312 ->
// 136, 439 -> 154; stride 2 on 8 x 96 x 224 x 224: forward 218 -> 144, weight
// gradient 236 -> 143; both gradients, 32 x 256 x 56 x 56, K = 63: 913 -> 271.
// What bounds them (stamped phases of NHWC 56 x 56, per plane and team): the
// walk takes 6.6 us of 14.5, with two waves per SIMD too few to hide the
// run starts' reloads; staging 4.2 and storing 2.7, where every lane of an
// NHWC access touches a cache line of its own; at stride 2, staging (four
// phases of strided rows).  Loading the next region ahead through registers
// was slower on NCHW (fewer resident workgroups) and no faster on NHWC.
#pragma once

#include "o1d_strip_kernels.h"
#include "o1d_walk.h"
#include "o1d_wave.h"

namespace o1d {
namespace walk {
namespace {

using strip::buffer_of;
using strip::kOob;
using strip::lds_addr;
using strip::lds_load;
using strip::lds_store;
using strip::Raw;

// The kernel's Params (every kernel's first argument) read afresh: the sizes
// a step needs are scalar loads at the step, instead of living in scalar
// registers (and, spilled, in vector registers) through the walks between.
__device__ __forceinline__ const Params& fresh_params() {
  auto p = (const __attribute__((address_space(4))) Params*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const Params*)p;
}

// ---------------------------------------------------------------- program

struct Prog {
  int* head;   // [0] transposed frame, [1] s, [2] finite angle, [4 + f] first chunk of phase f
  int* cnt;    // cells of a chunk
  int* brk;    // bit i: cell i of the chunk starts a run
  int* rb;     // run offset of a cell in bytes: 4 (a' S + b' - i (S + s)), i its index in the chunk
  float* w;    // weight of a cell
  int* bmin;   // per row of the line: its first column
  int* ent;    // per row and chain: the cell's place in rb, -1 without one
  __device__ __forceinline__ Prog(float* smem, const Params& P, int team) {
    head = reinterpret_cast<int*>(smem + team * P.prog_words);
    cnt = head + kProgHead;
    brk = cnt + P.maxch;
    rb = brk + P.maxch;
    w = reinterpret_cast<float*>(rb + kCell * P.maxch);
    bmin = rb + 2 * kCell * P.maxch;
    ent = bmin + 64;
  }
};

// The channel's line in its staging frame: rr and cc are the row and column
// of tap offset j = k - K / 2 before rounding.
struct Line {
  double cr, cc;
  bool tr, fin;
  __device__ __forceinline__ explicit Line(float theta) {
    fin = isfinite(theta);
    double s, c;
    sincos(fin ? (double)theta * kDegToRad : 0.0, &s, &c);
    tr = fabs(c) > fabs(s);
    cr = tr ? c : -s;
    cc = tr ? -s : c;
  }
};

// One tap's base cell and corner coefficients (rounding down: one corner).
struct Tap {
  int r, c;
  double fr, fc;
  __device__ __forceinline__ Tap(const Line& ln, int j, int mode) {
    const double rr = (double)j * ln.cr, cc = (double)j * ln.cc;
    r = floor_snapped(rr);
    c = floor_snapped(cc);
    fr = mode ? frac_snapped(rr, r) : 0.0;
    fc = mode ? frac_snapped(cc, c) : 0.0;
  }
  __device__ __forceinline__ double coef(int s, int t) const { return (s ? fr : 1.0 - fr) * (t ? fc : 1.0 - fc); }
};

// Builds the program of a channel with one wave, whose lane k holds tap k's
// weight wk.  Lane r holds row a = r - K / 2 of the line (K + mode <= 64
// rows).  A row's cells come from at most four taps (the line advances by at
// least 0.707 rows per tap) and lie within four columns (it moves at most
// one column per row).
template <int S>
__device__ void build_prog(const Params& P, const Prog& pg, float theta, float wk) {
  const int lane = threadIdx.x & 63;
  const int K = P.K, pad = K >> 1, str = P.str;
  const Line ln(theta);
  for (int i = lane; i < P.maxch; i += 64) {
    pg.brk[i] = 0;
    pg.cnt[i] = 0;
  }
  const int a = lane - pad;
  const bool row = lane < K + P.mode;
  double ws[4] = {0.0, 0.0, 0.0, 0.0};
  int b0 = 1 << 20;
  unsigned have = 0;
  const int jc = (int)floor((double)a / ln.cr);
  constexpr int kTaps = 6;  // tap offsets jc - 2 .. jc + 3
  int col[kTaps];
  float wt[kTaps];
  double c0[kTaps], c1[kTaps];  // coefficients at the tap's column and the next (0: not this row's)
#pragma unroll
  for (int d = 0; d < kTaps; ++d) {
    const int j = jc + d - 2;
    const Tap tp(ln, j, P.mode);
    const int s = a - tp.r;
    const bool in = row && j >= -pad && j <= K - 1 - pad && s >= 0 && s <= P.mode;
    col[d] = tp.c;
    wt[d] = __shfl(wk, (j + pad) & 63, 64);
    const double cr = in ? (s ? tp.fr : 1.0 - tp.fr) : 0.0;
    c0[d] = cr * (1.0 - tp.fc);
    c1[d] = cr * tp.fc;
    if (c0[d] != 0.0) b0 = min(b0, col[d]);
    if (c1[d] != 0.0) b0 = min(b0, col[d] + 1);
  }
#pragma unroll
  for (int d = 0; d < kTaps; ++d)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const double cf = t ? c1[d] : c0[d];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (cf != 0.0 && col[d] + t - b0 == u) {
          ws[u] += (double)wt[d] * cf;
          have |= 1u << u;
        }
    }
  // per chain: phase, cell on the phase's lattice
  const int Hs = ln.tr ? P.Q : P.P, Ws = ln.tr ? P.P : P.Q;
  int ca[4], cb[4], ph[4];
  int qa = a, fa = 0;
  if (str > 1) {
    qa = (a + 64 * str) / str - 64;
    fa = a - qa * str;
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int b = b0 + u;
    int qb = b, fb = 0;
    if (str > 1) {
      qb = (b + 64 * str) / str - 64;
      fb = b - qb * str;
    }
    ca[u] = P.sign * qa;
    cb[u] = P.sign * qb;
    const bool in = ((have >> u) & 1u) && ca[u] > -Hs && ca[u] < Hs && cb[u] > -Ws && cb[u] < Ws;
    ph[u] = in ? (ln.tr ? fb * str + fa : fa * str + fb) : -1;
  }
  // places in walk order: phases, chains, rows of increasing a'; the column
  // step from the predecessor in the chain where that is one row back
  int pos[4], chunk[4], step[4];
  int first = 0, nz = 0, np = 0, nm = 0;
  const int nchain = P.mode ? 4 : 2;
  for (int f = 0; f < P.nph; ++f) {
    int n = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (u >= nchain) continue;
      const bool in = ph[u] == f;
      const uint64_t m = __ballot(in);
      const uint64_t before = P.sign > 0 ? strip::below_mask(lane) : strip::above_mask(lane);
      const int pl = P.sign > 0 ? strip::hibit(m & before) : strip::lobit(m & before);
      const bool hp = in && pl >= 0 && pl < 64;
      const int pa = __shfl(ca[u], hp ? pl : lane, 64), pb = __shfl(cb[u], hp ? pl : lane, 64);
      const bool next = hp && ca[u] - pa == 1;
      const int db = cb[u] - pb;
      nz += strip::popc(__ballot(next && db == 0));
      np += strip::popc(__ballot(next && db == 1));
      nm += strip::popc(__ballot(next && db == -1));
      if (in) {
        pos[u] = n + strip::popc(m & before);
        chunk[u] = first;
        step[u] = next ? db : 99;
      }
      n += strip::popc(m);
    }
    const int nch = (n + kCell - 1) / kCell;
    if (lane == 0) pg.head[4 + f] = first;
    if (lane < nch) pg.cnt[first + lane] = min(kCell, n - kCell * lane);
    first += nch;
  }
  int s = 0;
  if (!P.small) s = np > nz && np >= nm ? 1 : (nm > nz && nm > np ? -1 : 0);
  if (lane == 0) {
    pg.head[4 + P.nph] = first;
    pg.head[0] = ln.tr ? 1 : 0;
    pg.head[1] = s;
    pg.head[2] = ln.fin ? 1 : 0;
  }
  if (P.op >= kWgrad) pg.bmin[lane] = b0;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    int e = -1;
    if (ph[u] >= 0) {
      const int i = pos[u] % kCell, m = chunk[u] + pos[u] / kCell;
      e = m * kCell + i;
      pg.rb[e] = 4 * (ca[u] * S + cb[u] - i * (S + s));
      pg.w[e] = ln.fin ? (float)ws[u] : __builtin_nanf("");
      if (i == 0 || step[u] != s) atomicOr(&pg.brk[m], (int)(1u << i));
    }
    if (P.op >= kWgrad) pg.ent[4 * lane + u] = e;
  }
}

// ---------------------------------------------------------------- geometry

// A workgroup's place: channel block, item range, partial row.
struct Work {
  int c0, item0, item1, run;
  __device__ __forceinline__ Work(const Params& P, int teams) {
    const int b = blockIdx.x;
    const int logical = P.xcd_per ? (b % 8) * P.xcd_per + b / 8 : b;
    run = logical / P.ncb;
    c0 = (logical - run * P.ncb) * teams;
    item0 = run * P.ipw;
    item1 = min(P.nitem, item0 + P.ipw);
  }
};

// Item: images n0 .. n0 + ng - 1, region origin (p0, q0) on the P x Q lattice.
struct Item {
  int n0, ng, p0, q0;
  __device__ __forceinline__ Item(const Params& P, int i) {
    const int nreg = P.nbh * P.nbw;
    const int grp = i / nreg, r = i - grp * nreg;
    n0 = grp * P.G;
    ng = min(P.G, P.N - n0);
    p0 = (r / P.nbw) * P.BH;
    q0 = (r % P.nbw) * P.BW;
  }
};

// Rows and columns (frame) of item i's region that lie in the plane.
struct Outputs {
  int h, w;
  __device__ __forceinline__ Outputs(const Params& P, int i, bool tr) {
    const Item it(P, i);
    const int p = min(P.BH, P.P - it.p0), q = min(P.BW, P.Q - it.q0);
    h = tr ? q : p;
    w = tr ? p : q;
  }
};

// A lattice view of a tensor: element (r, c) of image n at byte
// n img + off0 + r row + c col from base; `bytes` bounds one image's (NCHW:
// one plane's) offsets and ncol its columns.  Rows past the plane's end and
// before its start fall outside the range and read zeros.
struct View {
  const char* base;
  size_t img;
  int bytes, off0, row, col, ncol;
};

// phase f of a tensor of Hh x Ww planes taken every st pixels
template <typename T, int L>
__device__ __forceinline__ View view_of(const Params& P, const void* t, int Hh, int Ww, int st, int f, int c0) {
  View v;
  const int es = (int)sizeof(T), pi = st > 1 ? f / st : 0, pj = st > 1 ? f - pi * st : 0;
  const int px = L == kNHWC ? P.C * es : es;
  v.img = (size_t)P.C * Hh * Ww * es;
  v.base = static_cast<const char*>(t) + (L == kNHWC ? 0 : (size_t)c0 * Hh * Ww * es);
  v.bytes = Hh * Ww * px;
  v.off0 = (pi * Ww + pj) * px + (L == kNHWC ? c0 * es : 0);
  v.row = st * Ww * px;
  v.col = st * px;
  v.ncol = (Ww - pj + st - 1) / st;
  return v;
}

template <typename T>
__device__ __forceinline__ float load1(__amdgpu_buffer_rsrc_t rs, uint32_t off);
template <>
__device__ __forceinline__ float load1<float>(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
}
template <>
__device__ __forceinline__ float load1<uint16_t>(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  return to_f32((uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, off, 0, 0));
}
// the stored bits as loaded, and their value
template <typename T>
__device__ __forceinline__ uint32_t load_bits(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  if constexpr (sizeof(T) == 4)
    return __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
  else
    return __builtin_amdgcn_raw_buffer_load_b16(rs, off, 0, 0);
}
template <typename T>
__device__ __forceinline__ float bits_to_f32(uint32_t b) {
  return __uint_as_float(sizeof(T) == 4 ? b : b << 16);
}
template <typename T>
__device__ __forceinline__ void store1(__amdgpu_buffer_rsrc_t rs, uint32_t off, float v);
template <>
__device__ __forceinline__ void store1<float>(__amdgpu_buffer_rsrc_t rs, uint32_t off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs, off, 0, 0);
}
template <>
__device__ __forceinline__ void store1<uint16_t>(__amdgpu_buffer_rsrc_t rs, uint32_t off, float v) {
  __builtin_amdgcn_raw_buffer_store_b16(from_f32<uint16_t>(v), rs, off, 0, 0);
}

// The frames of the workgroup's channels and its tiles' LDS addresses.
template <int NT>
struct Tiles {
  uint32_t base[NT];  // LDS byte address of tile word kGuard of each team
  int tr[NT];
  int nch;            // channels that exist
  uint32_t trash;     // this lane's trash word
};

// Lanes of a wave over the next columns of a rectangle of which `rem` remain:
// 2^l2 columns per row, 64 / 2^l2 rows at once.  A remainder well below a
// power of two takes narrower pieces, so that few lanes are idle.
struct Lanes {
  int l2, lr, lc;
  __device__ __forceinline__ explicit Lanes(int rem) {
    l2 = rem > 44 ? 6 : (rem > 22 ? 5 : (rem > 10 ? 4 : 3));
    const int lane = threadIdx.x & 63;
    lr = lane >> l2;
    lc = lane & ((1 << l2) - 1);
  }
  __device__ __forceinline__ int rows() const { return 64 >> l2; }
  __device__ __forceinline__ int cols() const { return 1 << l2; }
};

// Small planes (NHWC): a plane is one step of the workgroup, so the batch in
// flight runs over the stacked planes.
template <typename T, int S, int NW>
struct SmallRect {
  int c, r, word[4];
  bool in;
  __device__ __forceinline__ SmallRect(const Params& P, const Tiles<4>& tl) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l2 = P.BW > 8 ? 4 : 3;  // 16 (8) lanes hold a row, the workgroup 16 (32) rows
    r = wave * (64 >> l2) + (lane >> l2);
    c = lane & ((1 << l2) - 1);
    in = c < P.BW && r < P.BH;
#pragma unroll
    for (int ch = 0; ch < 4; ++ch) word[ch] = tl.tr[ch] ? (P.halo + c) * S + P.ml + r : (P.halo + r) * S + P.ml + c;
  }
};

template <typename T, int S, int NW>
__device__ __forceinline__ void stage_small(const Params& P, const Tiles<4>& tl, const View& v, const Item& it) {
  constexpr int U = 4;
  const SmallRect<T, S, NW> rc(P, tl);
  const uint32_t off = rc.in && rc.c < v.ncol ? (uint32_t)(v.off0 + rc.c * v.col + rc.r * v.row) : kOob;
  for (int g0 = 0; g0 < P.G; g0 += U) {
    float e[U][4];
    if (P.vec && tl.nch == 4) {
      uint32_t raw[U][Raw<T>::kWords];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int g = g0 + u;
        Raw<T>::load(buffer_of(v.base + (size_t)(it.n0 + (g < it.ng ? g : 0)) * v.img, g < it.ng ? v.bytes : 0), off,
                     raw[u]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) e[u][ch] = Raw<T>::elem(raw[u], ch);
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int g = g0 + u;
        const __amdgpu_buffer_rsrc_t rs =
            buffer_of(v.base + (size_t)(it.n0 + (g < it.ng ? g : 0)) * v.img, g < it.ng ? v.bytes : 0);
#pragma unroll
        for (int ch = 0; ch < 4; ++ch)
          e[u][ch] = load1<T>(rs, ch < tl.nch ? off + (uint32_t)(ch * (int)sizeof(T)) : kOob);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int ch = 0; ch < 4; ++ch)
        lds_store(rc.in && g0 + u < P.G ? tl.base[ch] + 4u * (uint32_t)((g0 + u) * P.PS + rc.word[ch]) : tl.trash,
                  e[u][ch]);
  }
}

template <typename T, int S, int NW>
__device__ __forceinline__ void unstage_small(const Params& P, const Tiles<4>& tl, const View& v, const Item& it) {
  constexpr int U = 4;
  const SmallRect<T, S, NW> rc(P, tl);
  const uint32_t off = rc.in && rc.c < v.ncol ? (uint32_t)(v.off0 + rc.c * v.col + rc.r * v.row) : kOob;
  for (int g0 = 0; g0 < it.ng; g0 += U) {
    float e[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int ch = 0; ch < 4; ++ch)
        e[u][ch] = lds_load(rc.in && g0 + u < P.G ? tl.base[ch] + 4u * (uint32_t)((g0 + u) * P.PS + rc.word[ch])
                                                  : tl.trash);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int g = g0 + u;
      if (g < it.ng) {
        const __amdgpu_buffer_rsrc_t rs = buffer_of(v.base + (size_t)(it.n0 + g) * v.img, v.bytes);
        if (P.vec && tl.nch == 4) {
          Raw<T>::store(rs, off, e[u]);
        } else {
#pragma unroll
          for (int ch = 0; ch < 4; ++ch)
            if (ch < tl.nch) store1<T>(rs, off + (uint32_t)(ch * (int)sizeof(T)), e[u][ch]);
        }
      }
    }
  }
}

// Stages region (p0, q0) of `v` for the item's images into the teams' tiles,
// with `m` != 0 the pixels around it within reach of the line: a wave takes
// rows, U of them in flight per lane.
template <typename T, int L, int S, int NW, int NT>
__device__ __forceinline__ void stage(const Params& P, const Tiles<NT>& tl, const View& v, const Item& it, int m) {
  constexpr int U = L == kNHWC ? 8 : 14;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int both = max(P.halo, P.bmax);
  const int mr = !m ? 0 : (L == kNHWC ? both : (tl.tr[0] ? P.bmax : P.halo));
  const int mc = !m ? 0 : (L == kNHWC ? both : (tl.tr[0] ? P.halo : P.bmax));
  const int nr = P.BH + 2 * mr, nc = P.BW + 2 * mc;
  for (int g = 0; g < P.G; ++g) {
    const __amdgpu_buffer_rsrc_t rs =
        buffer_of(v.base + (size_t)(it.n0 + (g < it.ng ? g : 0)) * v.img, g < it.ng ? v.bytes : 0);
    for (int ck = 0; ck < nc;) {
      const Lanes ln(nc - ck);
      const int rs0 = NW * ln.rows();  // rows per step of the workgroup
      const int r0 = wave * ln.rows() + ln.lr;
      const int dv = rs0 * v.row;
      const int cx = ck + ln.lc, c = cx - mc, j = it.q0 + c;
      const bool in = cx < nc;
      const bool colok = in && j >= 0 && j < v.ncol;
      uint32_t off = colok ? (uint32_t)(v.off0 + j * v.col + (it.p0 + r0 - mr) * v.row) : kOob;
      uint32_t la[NT];
      int dl[NT];
      // the rectangle's rows that each tile holds (none for a column that it
      // does not hold; NHWC rectangles cover both frames)
      int row[NT];
      uint32_t cnt[NT];
#pragma unroll
      for (int ch = 0; ch < NT; ++ch) {
        const int word = tl.tr[ch] ? (P.halo + c) * S + P.ml + r0 - mr : (P.halo + r0 - mr) * S + P.ml + c;
        la[ch] = tl.base[ch] + 4u * (uint32_t)(g * P.PS + word);
        dl[ch] = 4 * rs0 * (tl.tr[ch] ? 1 : S);
        const int rm = !m ? 0 : (tl.tr[ch] ? P.bmax : P.halo), cm = !m ? 0 : (tl.tr[ch] ? P.halo : P.bmax);
        row[ch] = r0 - mr + rm;
        cnt[ch] = in && c >= -cm && c < P.BW + cm ? (uint32_t)(P.BH + 2 * rm) : 0u;
      }
      for (int k0 = 0; k0 * rs0 < nr; k0 += U) {
        if constexpr (L == kNCHW) {
          uint32_t e[U];
#pragma unroll
          for (int u = 0; u < U; ++u) e[u] = load_bits<T>(rs, off + (uint32_t)(u * dv));
#pragma unroll
          for (int u = 0; u < U; ++u)
            lds_store((uint32_t)(row[0] + u * rs0) < cnt[0] ? la[0] + (uint32_t)(u * dl[0]) : tl.trash,
                      bits_to_f32<T>(e[u]));
        } else {
          float e[U][4];
          if (P.vec && tl.nch == 4) {
            uint32_t raw[U][Raw<T>::kWords];
#pragma unroll
            for (int u = 0; u < U; ++u) Raw<T>::load(rs, off + (uint32_t)(u * dv), raw[u]);
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
              for (int ch = 0; ch < 4; ++ch) e[u][ch] = Raw<T>::elem(raw[u], ch);
          } else {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
              for (int ch = 0; ch < 4; ++ch)
                e[u][ch] = load1<T>(rs, ch < tl.nch ? off + (uint32_t)(u * dv + ch * (int)sizeof(T)) : kOob);
          }
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int ch = 0; ch < NT; ++ch)
              lds_store((uint32_t)(row[ch] + u * rs0) < cnt[ch] ? la[ch] + (uint32_t)(u * dl[ch]) : tl.trash, e[u][ch]);
        }
        off += (uint32_t)(U * dv);
#pragma unroll
        for (int ch = 0; ch < NT; ++ch) {
          la[ch] += (uint32_t)(U * dl[ch]);
          row[ch] += U * rs0;
        }
      }
      ck += ln.cols();
    }
  }
}

// Stores the tiles' region (p0, q0) to `v` (the range check drops rows past
// the plane).
template <typename T, int L, int S, int NW, int NT>
__device__ __forceinline__ void unstage(const Params& P, const Tiles<NT>& tl, const View& v, const Item& it) {
  constexpr int U = L == kNHWC ? 4 : 14;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int BH = P.BH, BW = P.BW;
  for (int g = 0; g < it.ng; ++g) {
    const __amdgpu_buffer_rsrc_t rs = buffer_of(v.base + (size_t)(it.n0 + g) * v.img, v.bytes);
    for (int ck = 0; ck < BW;) {
      const Lanes ln(BW - ck);
      const int rs0 = NW * ln.rows();
      const int r0 = wave * ln.rows() + ln.lr;
      const int dv = rs0 * v.row;
      const int c = ck + ln.lc, j = it.q0 + c;
      const bool colok = c < BW && j < v.ncol;
      uint32_t off = (uint32_t)(v.off0 + j * v.col + (it.p0 + r0) * v.row);
      uint32_t la[NT];
      int dl[NT];
      int row = r0;
#pragma unroll
      for (int ch = 0; ch < NT; ++ch) {
        const int word = tl.tr[ch] ? (P.halo + c) * S + P.ml + r0 : (P.halo + r0) * S + P.ml + c;
        la[ch] = tl.base[ch] + 4u * (uint32_t)(g * P.PS + word);
        dl[ch] = 4 * rs0 * (tl.tr[ch] ? 1 : S);
      }
      for (int k0 = 0; k0 * rs0 < BH; k0 += U) {
        float e[U][NT];
        // (rows past the region read the tile's other rows and are not stored)
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int ch = 0; ch < NT; ++ch) e[u][ch] = lds_load(la[ch] + (uint32_t)(u * dl[ch]));
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const uint32_t o = colok && row + u * rs0 < BH ? off + (uint32_t)(u * dv) : kOob;
          if constexpr (L == kNCHW) {
            store1<T>(rs, o, e[u][0]);
          } else if (P.vec && tl.nch == 4) {
            Raw<T>::store(rs, o, e[u]);
          } else {
#pragma unroll
            for (int ch = 0; ch < NT; ++ch)
              if (ch < tl.nch) store1<T>(rs, o + (uint32_t)(ch * (int)sizeof(T)), e[u][ch]);
          }
        }
        off += (uint32_t)(U * dv);
        row += U * rs0;
#pragma unroll
        for (int ch = 0; ch < NT; ++ch) la[ch] += (uint32_t)(U * dl[ch]);
      }
      ck += ln.cols();
    }
  }
}

// A lane's block: plane g of the item, frame rows b0 .. b0 + R - 1, strip
// columns j0 .. j0 + NC - 1, the LDS address of its first output.  Lanes
// without a task read a real block's addresses.
struct Block {
  int g, b0, j0, Hs, Ws;
  bool task, full;  // the lane has a block; the block lies inside the region
  uint32_t lb;
};

template <int S, int R, int NC, int SD, int LANES>
__device__ __forceinline__ Block block_of(const Params& P, int t, bool tr, uint32_t base) {
  Block bk;
  bk.Hs = tr ? P.BW : P.BH;
  bk.Ws = tr ? P.BH : P.BW;
  const Shape sh = shape_of(bk.Hs, bk.Ws, R, NC, SD, LANES);
  const int g = t / sh.ppt, r = t - g * sh.ppt;
  int band, cg;
  if (sh.dense) {
    band = r / sh.lpb;
    cg = r - band * sh.lpb;
  } else {
    const int blk = r >> 5, bb = blk / sh.bq;
    cg = 8 * (blk - bb * sh.bq) + (r & 7);
    band = 4 * bb + ((r >> 3) & 3);
  }
  const bool in = g < P.G && band < sh.nb;
  bk.task = in && cg < sh.ncg;
  bk.g = in ? g : 0;
  bk.b0 = in ? band * R : 0;
  bk.j0 = in ? sh.jlo + min(cg, sh.ncg - 1) * NC : sh.jlo;
  bk.lb = base + 4u * (uint32_t)(bk.g * P.PS + (P.halo + bk.b0) * S + P.ml + bk.j0);
  const int cmin = bk.j0 + (SD < 0 ? -(R - 1) : 0), cmax = bk.j0 + NC - 1 + (SD > 0 ? R - 1 : 0);
  bk.full = bk.task && bk.b0 + R <= bk.Hs && cmin >= 0 && cmax < bk.Ws;
  if (!bk.task) bk.b0 = bk.Hs;  // no position inside
  return bk;
}

// One chunk's program values: cell count and run bits (uniform), run offsets
// and weights (cell i in lane i).
struct Chunk {
  int n;
  uint32_t bits, vrb, vw;
  __device__ __forceinline__ Chunk(const Prog& pg, int m) {
    const int l = threadIdx.x & (kCell - 1);
    n = __builtin_amdgcn_readfirstlane(pg.cnt[m]);
    bits = (uint32_t)__builtin_amdgcn_readfirstlane(pg.brk[m]);
    vrb = (uint32_t)pg.rb[m * kCell + l];
    vw = __float_as_uint(pg.w[m * kCell + l]);
  }
};

// A team's walk for strips (R, NC, SD).
template <int S, int R_, int NC_, int SD_, int LANES_>
struct Steps {
  static constexpr int R = R_, NC = NC_, SD = SD_, LANES = LANES_, ST = S + SD_;
  static constexpr int NA = R * NC;
  // a block's values, row after row
  typedef float Vals[NA];
  typedef float Grid[R][NC];
  static __device__ __forceinline__ Grid& grid(Vals& v) { return reinterpret_cast<Grid&>(v); }
  static __device__ __forceinline__ Block block(const Params& P, int t, bool tr, uint32_t base) {
    return block_of<S, R, NC, SD, LANES>(P, t, tr, base);
  }
  // f(cell) for the chunk's cells, each behind its own uniform test (the
  // count passes through an empty asm statement, so that the test stays one
  // scalar compare)
  template <class F>
  static __device__ __forceinline__ void cells(int n, F&& f) {
    strip::static_for<kCell>([&](auto cc) __attribute__((always_inline)) {
      int nn = n;
      asm volatile("" : "+s"(nn));
      if (decltype(cc)::value < nn) f(cc);
    });
  }
  static __device__ __forceinline__ void gather(const Chunk& ch, uint32_t lb, Vals& acc) {
    float sl[R + 1][NC];
    uint32_t base = lb;
    cells(ch.n, [&](auto cc) __attribute__((always_inline)) {
      strip::gather_cell<R, NC, ST, decltype(cc)::value, kCell>(sl, base, lb, ch.vrb, ch.bits, ch.vw, grid(acc));
    });
  }
  static __device__ __forceinline__ void sums(const Chunk& ch, uint32_t lb, Vals& dv, float (&acc)[kCell]) {
    float sl[R + 1][NC];
    uint32_t base = lb;
    cells(ch.n, [&](auto cc) __attribute__((always_inline)) {
      strip::wgrad_cell<R, NC, ST, decltype(cc)::value, kCell>(sl, base, lb, ch.vrb, ch.bits, grid(dv), acc);
    });
  }
  static __device__ __forceinline__ void both(const Chunk& ch, uint32_t lb, Vals& xv, Vals& out,
                                              float (&acc)[kCell]) {
    float sl[R + 1][NC];
    uint32_t base = lb;
    cells(ch.n, [&](auto cc) __attribute__((always_inline)) {
      strip::bwd_cell<R, NC, ST, decltype(cc)::value, kCell, kCell>(sl, base, lb, ch.vrb, ch.bits, ch.vw, grid(xv),
                                                                   grid(out), acc);
    });
  }
  // Cell i's sum over the block's positions that hold outputs (frame rows below
  // hv, columns below wv) alone.
  static __device__ __forceinline__ float sum_inside(const Chunk& ch, int i, const Block& blk, const Vals& dv, int hv,
                                                     int wv) {
    const Block bk = fresh(blk);
    const uint32_t a = bk.lb + (uint32_t)__builtin_amdgcn_readlane((int)ch.vrb, i) + 4u * (uint32_t)(i * ST);
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        const float x = lds_load(a + 4u * (uint32_t)(r * ST + k));
        if (bk.b0 + r < hv && (unsigned)(bk.j0 + SD * r + k) < (unsigned)wv) s = fmaf(dv[r * NC + k], x, s);
      }
    return s;
  }
  // The block's positions (opaque to the optimiser: the tests of a ragged
  // block do not change from item to item, and hoisted out of the item loop
  // they would hold a mask per position).
  static __device__ __forceinline__ void take(const Block& blk, Vals& v) {
    const Block bk = fresh(blk);
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int k = 0; k < NC; ++k) v[i * NC + k] = lds_load(bk.lb + 4u * (uint32_t)(i * ST + k));
    if (!bk.full) {
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int k = 0; k < NC; ++k) v[i * NC + k] = inside(bk, i, k) ? v[i * NC + k] : 0.f;
    }
  }
  static __device__ __forceinline__ void put(const Block& blk, uint32_t trash, const Vals& v) {
    const Block bk = fresh(blk);
    if (bk.full) {
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int k = 0; k < NC; ++k) lds_store(bk.lb + 4u * (uint32_t)(i * ST + k), v[i * NC + k]);
    } else {
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int k = 0; k < NC; ++k)
          lds_store(inside(bk, i, k) ? bk.lb + 4u * (uint32_t)(i * ST + k) : trash, v[i * NC + k]);
    }
  }
  static __device__ __forceinline__ Block fresh(const Block& blk) {
    Block bk = blk;
    bk.b0 = (int)strip::opaque((uint32_t)blk.b0);
    bk.j0 = (int)strip::opaque((uint32_t)blk.j0);
    bk.lb = strip::opaque(blk.lb);
    return bk;
  }
  // position (i, k) of the block lies inside the region
  static __device__ __forceinline__ bool inside(const Block& bk, int i, int k) {
    const int col = bk.j0 + SD * i + k;
    return bk.b0 + i < bk.Hs && (unsigned)col < (unsigned)bk.Ws;
  }
};

// f(Steps<shape of the team's strip step s>()): the branch is uniform per
// wave, and every shape's path holds the same barriers.
template <int S, bool SMALL, class F>
__device__ __forceinline__ void with_shape(int s, F&& f) {
  if constexpr (SMALL) {
    f(Steps<S, kSmall, 1, 0, 64>());
  } else {
    if (s == 0)
      f(Steps<S, 28, 1, 0, 128>());
    else if (s > 0)
      f(Steps<S, 7, 4, 1, 128>());
    else
      f(Steps<S, 7, 4, -1, 128>());
  }
}

// What every kernel of the family sets up: zeroed tiles (margins stay zero)
// and sums, the teams' programs, the lanes' blocks.
template <typename T, int L, int S, bool SMALL>
struct Setup {
  static constexpr int NT = L == kNHWC ? 4 : 1, LANES = SMALL ? 64 : 128, NW = NT * LANES / 64, NA = SMALL ? kSmall : 28;
  Work wk;
  int team, t, c, s;
  bool live;  // the team's channel exists
  Prog pg;
  Tiles<NT> tl;
  bool tr;
  uint32_t base;  // LDS byte address of the team's tile
  float theta;
  __device__ __forceinline__ Setup(const Params& P, float* smem, const T* wgt, const float* angles)
      : wk(P, NT),
        team(__builtin_amdgcn_readfirstlane(threadIdx.x / LANES)),
        t(threadIdx.x % LANES),
        c(wk.c0 + team),
        live(c < P.C),
        pg(smem, P, team) {
    const int cc = min(c, P.C - 1);
    theta = angles[cc];
    const float w = wgt && t < P.K ? to_f32(wgt[(size_t)cc * P.K + t]) : 0.f;
    float4* z = reinterpret_cast<float4*>(smem + P.tile_off);
    const int n4 = (P.words - P.tile_off) >> 2;
    for (int i = threadIdx.x; i < n4; i += 64 * NW) z[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (t < 64) build_prog<S>(P, pg, theta, w);
    __syncthreads();
    s = __builtin_amdgcn_readfirstlane(pg.head[1]);
#pragma unroll
    for (int ch = 0; ch < NT; ++ch) {
      tl.base[ch] = lds_addr(smem + P.tile_off + ch * P.tile_words + kGuard);
      tl.tr[ch] = __builtin_amdgcn_readfirstlane(Prog(smem, P, ch).head[0]);
    }
    tl.nch = min(NT, P.C - wk.c0);
    tl.trash = lds_addr(smem + P.trash_off + (threadIdx.x & 63));
    tr = __builtin_amdgcn_readfirstlane(pg.head[0]) != 0;
    base = lds_addr(smem + P.tile_off + team * P.tile_words + kGuard);
  }
  __device__ __forceinline__ bool finite() const { return __builtin_amdgcn_readfirstlane(pg.head[2]) != 0; }
  __device__ __forceinline__ int first(int f) const { return __builtin_amdgcn_readfirstlane(pg.head[4 + f]); }
  // Item i's region of the view (view(P): the tensor's lattice view) into the tiles.
  template <class V>
  __device__ __forceinline__ void fill(V&& view, int i, bool margins) const {
    const Params& P = fresh_params();
    if constexpr (SMALL)
      stage_small<T, S, NW>(P, tl, view(P), Item(P, i));
    else
      stage<T, L, S, NW, NT>(P, tl, view(P), Item(P, i), margins ? P.banded : 0);
    __syncthreads();
  }
  // The tiles' region of item i out to the view.
  template <class V>
  __device__ __forceinline__ void drain(V&& view, int i) const {
    const Params& P = fresh_params();
    if constexpr (SMALL)
      unstage_small<T, S, NW>(P, tl, view(P), Item(P, i));
    else
      unstage<T, L, S, NW, NT>(P, tl, view(P), Item(P, i));
    __syncthreads();
  }
};

template <int A>
__device__ __forceinline__ void clear(float (&a)[A]) {
#pragma unroll
  for (int i = 0; i < A; ++i) a[i] = 0.f;
}

template <int A>
__device__ __forceinline__ void poison(float (&a)[A]) {
#pragma unroll
  for (int i = 0; i < A; ++i) a[i] = __builtin_nanf("");
}

// ---------------------------------------------------------------- gather

// Forward pass (source phases added up) and input gradient (one output
// phase at a time).  A barrier separates staging, walk, the blocks' writes
// into the tile and the tile's store; workgroups that share a CU cover each
// other's latencies.
template <typename T, int L, int S, bool SMALL>
__global__ __launch_bounds__((L == kNHWC ? 4 : 1) * (SMALL ? 64 : 128)) __attribute__((
    amdgpu_waves_per_eu(L == kNHWC ? 2 : 4))) void walk_gather(Params P, const T* __restrict__ in,
                                                              const T* __restrict__ wgt,
                                                              const float* __restrict__ theta, T* __restrict__ out) {
  extern __shared__ float smem[];
  using St = Setup<T, L, S, SMALL>;
  const St st(P, smem, wgt, theta);
  const bool fwd = P.op == kFwd;
  const int c0 = st.wk.c0;
  with_shape<S, SMALL>(st.s, [&](auto sp) __attribute__((always_inline)) {
    const Block bk = sp.block(P, st.t, st.tr, st.base);
    typename decltype(sp)::Vals acc;
    for (int i = st.wk.item0; i < st.wk.item1; ++i) {
      const int nph = fresh_params().nph;
      for (int f = 0; f < nph; ++f) {
        st.fill([&](const Params& Q) __attribute__((always_inline)) {
          return fwd ? view_of<T, L>(Q, in, Q.H, Q.W, Q.str, f, c0) : view_of<T, L>(Q, in, Q.P, Q.Q, 1, 0, c0);
        }, i, true);
        if (!fwd || f == 0) clear(acc);
        for (int m = st.first(f); m < st.first(f + 1); ++m) sp.gather(Chunk(st.pg, m), bk.lb, acc);
        // a non-finite angle poisons every output: through its cells' weights,
        // and here in a phase without cells (tested first: a read of `finite`
        // for every item cost the NHWC gathers 3%)
        if (st.first(f) == st.first(f + 1) && !st.finite()) poison(acc);
        __syncthreads();  // the tiles are free
        if (!fwd || f == nph - 1) {
          sp.put(bk, st.tl.trash, acc);
          __syncthreads();  // the outputs are in the tiles
          st.drain([&](const Params& Q) __attribute__((always_inline)) {
            return fwd ? view_of<T, L>(Q, out, Q.P, Q.Q, 1, 0, c0) : view_of<T, L>(Q, out, Q.H, Q.W, Q.str, f, c0);
          }, i);
        }
      }
    }
  });
}

// ---------------------------------------------------------------- weight gradients

// Adds the wave's per-cell sums of chunk m into its own row of LDS sums.  A
// lane's chain is one item, at most 28 products long, and the sums of the
// chains are kept in doubles: one float chain over a workgroup's items had an
// error of 2.5e-7 in 64 x 96 x 56 x 56 (NHWC, K = 31), chains of 56 products
// 1.6e-7 (times unchanged).
//
// Strips reach past the region and lanes without a task walk a real block, all
// times a zero, which an infinite or NaN pixel turns into NaN.  A cell whose
// sum is not finite is therefore summed again over the item's outputs alone
// (`again(cell)`: this lane's share), so that it is what its pixels make it.
template <class F>
__device__ __forceinline__ void flush(float (&acc)[kCell], double* sums, int m, F&& again) {
  const int lane = threadIdx.x & 63;
  float v = wave::sum32<0>(acc);
  for (uint64_t bad = __ballot(!isfinite(v)); bad != 0;) {
    const int i = (strip::lobit(bad) >> 1) & (kCell - 1);
    const float t = strip::wave_sum(again(i));
    if (((lane >> 1) & (kCell - 1)) == i) v = t;
    bad &= ~(3ull << (2 * i));
  }
  if ((lane & 1) == 0) sums[m * kCell + ((lane >> 1) & (kCell - 1))] += v;
  clear(acc);
}

// partial[(run C + c) K + k]: the team's cell sums folded into its taps
// (coefficient times sum, corners and waves in a fixed order).
template <class St>
__device__ __forceinline__ void fold(const Params& P, const St& st, const double* sums, float* partial) {
  __syncthreads();
  if (!st.live || st.t >= P.K) return;
  const Line ln(st.theta);
  const int pad = P.K >> 1;
  const Tap tp(ln, st.t - pad, P.mode);
  double v = 0.0;
  for (int s = 0; s <= P.mode; ++s)
    for (int u = 0; u <= P.mode; ++u) {
      const double cf = tp.coef(s, u);
      if (cf == 0.0) continue;
      const int r = tp.r + s + pad;
      const int e = st.pg.ent[4 * r + tp.c + u - st.pg.bmin[r]];
      if (e < 0) continue;
      double x = 0.0;
      for (int w = 0; w < St::LANES / 64; ++w) x += sums[w * P.maxch * kCell + e];
      v += cf * x;
    }
  partial[((size_t)st.wk.run * P.C + st.c) * P.K + st.t] = ln.fin ? (float)v : __builtin_nanf("");
}

// Weight gradient: dy of the region in registers, x walked phase by phase.
template <typename T, int L, int S, bool SMALL>
__global__ __launch_bounds__((L == kNHWC ? 4 : 1) * (SMALL ? 64 : 128)) __attribute__((
    amdgpu_waves_per_eu(L == kNHWC ? 2 : 3))) void walk_wgrad(Params P, const T* __restrict__ x,
                                                             const T* __restrict__ dy, const float* __restrict__ theta,
                                                             float* __restrict__ partial) {
  extern __shared__ float smem[];
  using St = Setup<T, L, S, SMALL>;
  const St st(P, smem, static_cast<const T*>(nullptr), theta);
  double* const team_sums = reinterpret_cast<double*>(smem + P.sum_off + st.team * P.sum_words);
  double* sums = team_sums + (st.t >> 6) * P.maxch * kCell;
  const int c0 = st.wk.c0;
  float acc[kCell];
  clear(acc);
  with_shape<S, SMALL>(st.s, [&](auto sp) __attribute__((always_inline)) {
    const Block bk = sp.block(P, st.t, st.tr, st.base);
    typename decltype(sp)::Vals dv;
    for (int i = st.wk.item0; i < st.wk.item1; ++i) {
      st.fill([&](const Params& Q) __attribute__((always_inline)) { return view_of<T, L>(Q, dy, Q.P, Q.Q, 1, 0, c0); },
              i, false);
      sp.take(bk, dv);
      __syncthreads();
      const int nph = fresh_params().nph;
      for (int f = 0; f < nph; ++f) {
        st.fill([&](const Params& Q) __attribute__((always_inline)) {
          return view_of<T, L>(Q, x, Q.H, Q.W, Q.str, f, c0);
        }, i, true);
        for (int m = st.first(f); m < st.first(f + 1); ++m) {
          sp.sums(Chunk(st.pg, m), bk.lb, dv, acc);
          flush(acc, sums, m, [&](int e) __attribute__((always_inline)) {
            const Outputs o(fresh_params(), i, st.tr);
            return sp.sum_inside(Chunk(st.pg, m), e, bk, dv, o.h, o.w);
          });
        }
        __syncthreads();
      }
    }
  });
  fold(P, st, team_sums, partial);
}

// Both gradients (NCHW, stride 1, rounded down): x of the region in
// registers, dy walked with the mirrored program; every window value feeds
// the lane's input-gradient block and the cell's sum.
template <typename T, int S>
__global__ __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(3))) void walk_bwd(
    Params P, const T* __restrict__ x, const T* __restrict__ dy, const T* __restrict__ wgt,
    const float* __restrict__ theta, T* __restrict__ dx, float* __restrict__ partial) {
  extern __shared__ float smem[];
  using St = Setup<T, kNCHW, S, false>;
  const St st(P, smem, wgt, theta);
  auto view = [&](const void* t) __attribute__((always_inline)) {
    return [=](const Params& Q) __attribute__((always_inline)) { return view_of<T, kNCHW>(Q, t, Q.H, Q.W, 1, 0, st.c); };
  };
  double* const team_sums = reinterpret_cast<double*>(smem + P.sum_off);
  double* sums = team_sums + (st.t >> 6) * P.maxch * kCell;
  const int nch = st.first(1);
  float acc[kCell];
  clear(acc);
  with_shape<S, false>(st.s, [&](auto sp) __attribute__((always_inline)) {
    const Block bk = sp.block(P, st.t, st.tr, st.base);
    typename decltype(sp)::Vals xv, out;
    for (int i = st.wk.item0; i < st.wk.item1; ++i) {
      st.fill(view(x), i, false);
      sp.take(bk, xv);
      __syncthreads();
      st.fill(view(dy), i, true);
      clear(out);
      for (int m = 0; m < nch; ++m) {
        sp.both(Chunk(st.pg, m), bk.lb, xv, out, acc);
        flush(acc, sums, m, [&](int e) __attribute__((always_inline)) {
          const Outputs o(fresh_params(), i, st.tr);
          return sp.sum_inside(Chunk(st.pg, m), e, bk, xv, o.h, o.w);
        });
      }
      __syncthreads();
      sp.put(bk, st.tl.trash, out);
      __syncthreads();
      st.drain(view(dx), i);
    }
  });
  fold(P, st, team_sums, partial);
}

// ---------------------------------------------------------------- launch

template <typename T, int L, int S, bool SMALL>
const void* gather_fn() { return reinterpret_cast<const void*>(walk_gather<T, L, S, SMALL>); }
template <typename T, int L, int S, bool SMALL>
const void* wgrad_fn() { return reinterpret_cast<const void*>(walk_wgrad<T, L, S, SMALL>); }
template <typename T, int S>
const void* bwd_fn() { return reinterpret_cast<const void*>(walk_bwd<T, S>); }

// NHWC: a pixel's four channels as one access, where every pixel's run starts
// on a 4-byte boundary (what 8- and 16-byte buffer accesses need) and the
// block has four channels.
template <typename T, int L>
Params with_vec(const Plan& pl, const void* a, const void* b) {
  Params p = pl.p;
  p.vec = L == kNHWC && ((uintptr_t)a | (uintptr_t)b | (uintptr_t)(p.C * sizeof(T))) % 4 == 0;
  return p;
}

template <typename T, int L, int S, bool SMALL>
hipError_t gather_launch(const Plan& pl, const void* in, const void* w, const float* theta, void* out,
                         hipStream_t stream) {
  const hipError_t e = strip::allow_full_lds<gather_fn<T, L, S, SMALL>>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((walk_gather<T, L, S, SMALL>), dim3((unsigned)pl.p.nblocks),
                     dim3((L == kNHWC ? 4 : 1) * (SMALL ? 64 : 128)), pl.lds_bytes, stream,
                     with_vec<T, L>(pl, in, out),
                     static_cast<const T*>(in), static_cast<const T*>(w), theta, static_cast<T*>(out));
  return hipGetLastError();
}

template <typename T, int L, int S, bool SMALL>
hipError_t wgrad_launch(const Plan& pl, const void* x, const void* dy, const float* theta, float* partial,
                        hipStream_t stream) {
  const hipError_t e = strip::allow_full_lds<wgrad_fn<T, L, S, SMALL>>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((walk_wgrad<T, L, S, SMALL>), dim3((unsigned)pl.p.nblocks),
                     dim3((L == kNHWC ? 4 : 1) * (SMALL ? 64 : 128)), pl.lds_bytes, stream,
                     with_vec<T, L>(pl, x, dy),
                     static_cast<const T*>(x), static_cast<const T*>(dy), theta, partial);
  return hipGetLastError();
}

template <typename T, int S>
hipError_t bwd_launch(const Plan& pl, const void* x, const void* dy, const void* w, const float* theta, void* dx,
                      float* partial, hipStream_t stream) {
  const hipError_t e = strip::allow_full_lds<bwd_fn<T, S>>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((walk_bwd<T, S>), dim3((unsigned)pl.p.nblocks), dim3(128), pl.lds_bytes, stream, pl.p,
                     static_cast<const T*>(x), static_cast<const T*>(dy), static_cast<const T*>(w), theta,
                     static_cast<T*>(dx), partial);
  return hipGetLastError();
}

template <typename T, int L>
hipError_t gather_t(const Plan& pl, const void* in, const void* w, const float* theta, void* out,
                    hipStream_t stream) {
  if constexpr (L == kNHWC)
    if (pl.S == kSmallS) return gather_launch<T, L, kSmallS, true>(pl, in, w, theta, out, stream);
#define O1D_CASE(SV) \
  if (pl.S == SV) return gather_launch<T, L, SV, false>(pl, in, w, theta, out, stream);
  O1D_WALK_STRIDES(O1D_CASE)
  if constexpr (L == kNCHW) {
    O1D_WALK_STRIDES_NCHW(O1D_CASE)
  }
#undef O1D_CASE
  return hipErrorInvalidValue;
}

template <typename T, int L>
hipError_t wgrad_t(const Plan& pl, const void* x, const void* dy, const float* theta, float* partial,
                   hipStream_t stream) {
  if constexpr (L == kNHWC)
    if (pl.S == kSmallS) return wgrad_launch<T, L, kSmallS, true>(pl, x, dy, theta, partial, stream);
#define O1D_CASE(SV) \
  if (pl.S == SV) return wgrad_launch<T, L, SV, false>(pl, x, dy, theta, partial, stream);
  O1D_WALK_STRIDES(O1D_CASE)
  if constexpr (L == kNCHW) {
    O1D_WALK_STRIDES_NCHW(O1D_CASE)
  }
#undef O1D_CASE
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t bwd_t(const Plan& pl, const void* x, const void* dy, const void* w, const float* theta, void* dx,
                 float* partial, hipStream_t stream) {
#define O1D_CASE(SV) \
  if (pl.S == SV) return bwd_launch<T, SV>(pl, x, dy, w, theta, dx, partial, stream);
  O1D_WALK_STRIDES(O1D_CASE)
  O1D_WALK_STRIDES_NCHW(O1D_CASE)
#undef O1D_CASE
  return hipErrorInvalidValue;
}

}  // namespace
}  // namespace walk
}  // namespace o1d
