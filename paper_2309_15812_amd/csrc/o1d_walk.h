// Host-side plan of the walk kernels: forward pass, input gradient, weight
// gradient and both gradients in one pass for either memory layout, stride
// 1 .. 3, either sampling, any plane size and K <= 63 (NHWC calls, and NCHW
// planes that the strip and plane kernels do not take, where `applies` says
// that they are faster than the table-driven general kernels).
//
// A team of 128 lanes (planes of at most 14 x 14: 64 lanes) works on one
// channel, with the register-blocked walks of the strip kernels.  NCHW
// workgroups hold one team, NHWC workgroups four, one per channel of a
// pixel's 16-byte (bfloat16: 8-byte) run, so that every global access moves
// the four channels together and each team's tile holds one channel's plane.
//
// Stride: the operation is split into str x str phases.  Source pixels
// (str i + pi, str j + pj) form phase (pi, pj), and on the phase's own
// lattice the taps that land on it are a stride-1 line; the forward pass and
// the weight gradient add the phases up, the input gradient runs one phase
// of its output at a time.  Every phase's tile has the size of the small
// plane P x Q, so nothing is staged twice and no lane works on zeros between
// lattice points.
//
// Large planes are cut into regions of BH x BW outputs, whose tiles hold the
// neighbouring pixels within reach of the line; a whole plane's tile keeps a
// zero margin instead, which stacked planes (G of them) and consecutive rows
// share.
#pragma once

#include <stddef.h>

#include "o1d_gen.h"
#include "o1d_launch.h"
#include "o1d_plan.h"

namespace o1d {
namespace walk {

constexpr int kMaxK = 63;      // one wave builds the program, a lane per row of the line
constexpr int kMaxStride = 3;
constexpr int kCell = 32;      // cells per chunk of a program
constexpr int kGuard = 16;
constexpr int kSmall = 14;     // planes up to kSmall x kSmall: one strip of 14 rows per column, one-wave teams
constexpr int kSmallS = 27;    // their tile's row stride (14 columns and a shared margin of 13)
constexpr int kProgHead = 64;  // program words before the per-chunk and per-cell arrays
constexpr long long kMaxPartBytes = 8 << 20;  // partial rows of a plain weight gradient: no more than o1d_bwd_noalloc holds
constexpr int kRowWords = 64 + 256;  // first column and four cell slots of every row of the line

// Odd tile row strides compiled into the kernels.  79 is the least that takes
// 56-column planes at K = 31 with bilinear sampling (a wider tile leaves four
// resident workgroups per CU instead of five).
// (Four NHWC tiles of stride 119 do not fit in LDS.)
#define O1D_WALK_STRIDES(X) X(51) X(63) X(79) X(87) X(103)
#define O1D_WALK_STRIDES_NCHW(X) X(119)
constexpr int kStrides[] = {51, 63, 79, 87, 103, 119};
constexpr int kMaxStrideNhwc = 103;

enum Op { kFwd = 0, kDgrad = 1, kWgrad = 2, kBwd = 3 };
enum Layout { kNCHW = 0, kNHWC = 1 };

__host__ __device__ inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// Lanes of a region of Hs x Ws outputs (staging frame) for the strip shape:
// R outputs per strip, NC adjacent strips per lane, steps (1, sd).  Vertical
// strips take one lane per column, band after band (a band's lanes rounded
// up to whole half-waves where that costs no plane, so that a half-wave reads
// consecutive columns); diagonal ones half-wave blocks of 8 column groups x 4
// bands (R = 7 rows apart at an odd row stride: 32 distinct banks), or one
// lane each, band after band, where the blocks would cost a plane.
struct Shape {
  int nb, nj, jlo, ncg, ppt, lpb, bq, dense;
};

__host__ __device__ inline Shape shape_of(int Hs, int Ws, int R, int NC, int sd, int lanes) {
  Shape t;
  t.nb = cdiv(Hs, R);
  t.nj = Ws + (sd ? R - 1 : 0);
  t.jlo = sd > 0 ? -(R - 1) : 0;
  t.ncg = cdiv(t.nj, NC);
  t.bq = cdiv(t.ncg, 8);
  const int blocked = 32 * t.bq * cdiv(t.nb, 4), one = t.nb * t.ncg;
  t.dense = !sd || lanes / one > lanes / blocked;
  t.lpb = t.ncg;
  if (t.dense) {
    const int planes = lanes / one;
    for (int a = 64; a >= 32; a /= 2) {
      const int l = cdiv(t.ncg, a) * a;
      if (planes >= 1 && t.nb * l <= lanes && lanes / (t.nb * l) == planes) {
        t.lpb = l;
        break;
      }
    }
  }
  t.ppt = t.dense ? t.nb * t.lpb : blocked;
  return t;
}

struct Params {
  int N, C, H, W, K;  // input plane H x W
  int P, Q;           // output plane of the stride: P = (H - 1) / str + 1
  int str, mode, op, sign, small;
  int nph;            // phases = str str
  int BH, BW, nbh, nbw, banded;  // region of outputs, regions along rows and columns, more than one region
  int G;              // planes per item (whole planes only)
  int ngrp;           // image groups = ceil(N / G)
  int nitem, ipw;     // items (image group, region); items per workgroup
  int runs;           // workgroups per channel block = ceil(nitem / ipw)
  int ncb;            // channel blocks
  int nblocks, xcd_per;
  int halo, bmax;     // rows and columns (frame) the line reaches beyond an output
  int ml;             // tile columns left of the region
  int PR, PS;         // tile rows and words from one stacked plane to the next
  int maxch;          // program chunks
  int vec;            // NHWC: a pixel's four channels move as one access (set at the launch)
  int prog_words, tile_words, sum_words;  // LDS words per team
  int tile_off, sum_off, trash_off, words;  // LDS word offsets (programs at 0) and total
};

struct Plan {
  Params p{};
  int S = 0;
  size_t lds_bytes = 0;
  size_t parts = 0;  // weight gradients: partial rows per channel (= runs)
  bool ok = false;
};

inline int out_size(int n, int str) { return (n - 1) / str + 1; }

// Resident workgroups per CU by LDS (granted in 1 KB steps out of slightly
// less than 160 KB) and by `waves` waves per workgroup at `per_simd` waves
// per SIMD.
inline int resident(size_t lds_bytes, int waves, int per_simd) {
  const int by_lds = (int)((kMaxLdsBytes - 512) / ((lds_bytes + 1023) / 1024 * 1024));
  const int by_regs = 4 * per_simd / waves;
  const int n = by_lds < by_regs ? by_lds : by_regs;
  return n < 1 ? 1 : n;
}

// Pixels staged around a region, and one item's staging of one phase: row
// steps and batches of loads in flight.
inline int margin_of(const Params& p) { return p.banded ? (p.halo > p.bmax ? p.halo : p.bmax) : 0; }
struct Staging {
  int slots, pieces;
};
inline Staging staging_of(const Params& p, int layout, int waves) {
  Staging s{0, 0};
  const int mg = margin_of(p);
  for (int c = p.BW + 2 * mg; c > 0;) {
    const int w = c > 44 ? 64 : (c > 22 ? 32 : (c > 10 ? 16 : 8)), st = cdiv(p.BH + 2 * mg, waves * (64 / w));
    s.slots += p.G * st;
    s.pieces += p.G * cdiv(st, layout == kNHWC ? 8 : 14);
    c -= w;
  }
  return s;
}

// esize: bytes per element.  (Alignment plays no part: NCHW accesses are
// single elements, and the NHWC launch looks at the addresses itself.)
inline Plan plan_walk(int op, int layout, int N, int C, int H, int W, int K, int str, int mode, int esize) {
  Plan best;
  if (N < 1 || C < 1 || H < 1 || W < 1 || K < 1 || K > kMaxK || str < 1 || str > kMaxStride) return best;
  if (op == kBwd && (layout != kNCHW || str != 1 || mode != 0)) return best;
  // byte offsets within a plane (NCHW) or an image (NHWC) stay well below 2^31
  const long long reach = (long long)(H + 4 * 64) * (W + 4 * 64) * (layout == kNHWC ? C : 1) * 4;
  if (reach >= (1ll << 30)) return best;
  Params q{};
  q.N = N; q.C = C; q.H = H; q.W = W; q.K = K;
  q.P = out_size(H, str);
  q.Q = out_size(W, str);
  q.str = str; q.mode = mode; q.op = op;
  q.sign = op == kDgrad || op == kBwd ? -1 : 1;
  q.nph = str * str;
  const int M0 = q.P > q.Q ? q.P : q.Q;
  q.small = layout == kNHWC && M0 <= kSmall ? 1 : 0;
  const int teams = layout == kNHWC ? 4 : 1;
  const int lanes = q.small ? 64 : 128;
  const int R = q.small ? kSmall : 28;
  // Reach on a phase's lattice.  The staging frame puts the line's longer
  // extent along its rows, so a cell's column offset is at most
  // floor((K / 2) sin 45 deg) + 1 in magnitude (one more kept for margin; one
  // more for bilinear corners); cells that reach no pixel of the plane from
  // any output are dropped.
  const int cap = M0 - 1;
  q.halo = cdiv(K / 2 + mode, str);
  if (q.halo > cap) q.halo = cap;
  q.bmax = cdiv((int)((K / 2) * 0.70711) + 2 + mode, str);
  if (q.bmax > cap) q.bmax = cap;
  const int maxcells = K * (mode ? 4 : 1);
  q.maxch = q.nph + maxcells / kCell;
  q.prog_words = kProgHead + 2 * q.maxch + 2 * kCell * q.maxch + (op >= kWgrad ? kRowWords : 0);
  q.prog_words = (q.prog_words + 3) & ~3;
  q.ncb = cdiv(C, teams);
  const int waves = teams * lanes / 64;
  q.sum_words = op >= kWgrad ? lanes / 64 * q.maxch * kCell * 2 : 0;  // doubles
  const int diag = q.small ? 0 : 9;  // columns a diagonal block spans beyond its first output
  double best_cost = 0.0;
  // region sides tried: the whole side, halves, thirds and quarters, and
  // sides of about two, one and a half, one and half a strip of 28
  int nhs[8], nws[8];
  auto sides = [](int n, int* out) {
    int m = 0;
    for (int nb : {1, 2, 3, 4, cdiv(n, 56), cdiv(n, 42), cdiv(n, 28), cdiv(n, 14)}) {
      bool seen = nb > n;
      for (int i = 0; i < m; ++i) seen = seen || out[i] == nb;
      if (!seen) out[m++] = nb;
    }
    return m;
  };
  const int mh = sides(q.P, nhs), mw = sides(q.Q, nws);
  for (int ih = 0; ih < mh; ++ih)
    for (int iw = 0; iw < mw; ++iw) {
      const int nbh = nhs[ih], nbw = nws[iw];
      if (q.small && nbh * nbw > 1) continue;
      Params p = q;
      p.BH = cdiv(q.P, nbh);
      p.BW = cdiv(q.Q, nbw);
      if (cdiv(q.P, p.BH) != nbh || cdiv(q.Q, p.BW) != nbw) continue;
      p.nbh = nbh;
      p.nbw = nbw;
      p.banded = nbh * nbw > 1;
      const int M = p.BH > p.BW ? p.BH : p.BW;
      // a whole plane's rows share one zero margin; a region has real pixels
      // within bmax columns on both sides of its rows
      const int need = p.banded ? M + 2 * p.bmax + diag + 6 : M + p.bmax + diag;
      p.ml = p.small ? p.bmax : (p.banded ? p.bmax + 6 : p.bmax + diag);
      int S = 0;
      if (p.small) {
        S = need <= kSmallS ? kSmallS : 0;
      } else {
        for (int s : kStrides)
          if (s >= need) {
            S = layout == kNCHW || s <= kMaxStrideNhwc ? s : 0;
            break;
          }
      }
      if (S == 0) continue;
      int ppt = 0, cover = 0;
      for (int f = 0; f < 2; ++f)
        for (int sd = 0; sd < (p.small ? 1 : 2); ++sd) {
          const int r = sd ? 7 : R;
          const Shape t = shape_of(f ? p.BW : p.BH, f ? p.BH : p.BW, r, sd ? 4 : 1, sd, lanes);
          if (t.ppt > ppt) ppt = t.ppt;
          if (t.nb * r > cover) cover = t.nb * r;
        }
      if (ppt > lanes) continue;
      p.PR = M + p.halo;
      p.PS = p.PR * S;
      if (p.small)  // planes of 14 columns side by side in the banks
        while (p.PS % 32 != 14) ++p.PS;
      p.trash_off = 64;  // one word per lane of a wave
      const int gmax = p.banded ? 1 : (lanes / ppt < N ? lanes / ppt : N);
      for (int G = gmax; G >= 1; --G) {
        p.G = G;
        // Idle rows of the last strips read past their tile's rows.  The
        // gathers drop what such lanes compute; the weight gradients multiply
        // it by zero, so their tiles are as long as the reads (the next
        // channel's pixels may be infinite).
        const int slack = (cover - M + 2) * S;
        p.tile_words = (kGuard + (p.halo + 1) * S + G * p.PS + 16 + (op >= kWgrad ? slack : 0) + 3) & ~3;
        p.tile_off = teams * p.prog_words;
        p.sum_off = p.tile_off + teams * p.tile_words;
        p.trash_off = p.sum_off + teams * p.sum_words;
        p.words = p.trash_off + 64;
        if (op < kWgrad && p.words < p.sum_off + slack) p.words = (p.sum_off + slack + 3) & ~3;
        const size_t lds = (size_t)p.words * 4;
        if (lds > kMaxLdsBytes - 1024 || p.words >= 65536) continue;
        // Time of a CU, in cycles.  An item's instructions per wave: staging
        // slots (an NHWC slot writes four tiles) and the store, the walk (28
        // products and a window row per cell; a bilinear line has about 2.4
        // cells per row); four cycles each on one of four SIMDs.  Alone it
        // also waits for each piece's loads (about 2500 cycles) and at
        // barriers; resident workgroups overlap that.
        const int res = resident(lds, waves, teams == 4 ? 2 : (op == kWgrad || op == kBwd ? 3 : 4));
        const int mg = margin_of(p), nr = p.BH + 2 * mg;
        const Staging sg = staging_of(p, layout, waves);
        const int pieces = sg.pieces, slots = sg.slots;
        const double per_slot = teams == 4 ? 20.0 : 6.0;
        const double instr = p.nph * slots * per_slot + cdiv(G * p.BH * p.BW, waves * 64) * per_slot + 200.0 +
                             K * (mode ? 2.4 : 1.0) * (p.small ? 22.0 : 36.0) + 60.0 * p.nph;
        const double alone = 6.0 * instr + p.nph * (2500.0 * pieces + 600.0) + 2000.0;
        // (bytes over about seven a cycle, the chip's 4.5 TB/s shared by its
        // CUs; a strided row of an NCHW phase moves all its columns)
        const double bytes = (p.nph * (double)nr * (p.BW + 2 * mg) * (layout == kNHWC ? 4 : str) +
                              (double)p.BH * p.BW * teams) * G * esize;
        double busy = instr * waves;
        if (bytes / 7.0 > busy) busy = bytes / 7.0;
        busy *= res;
        const long long nit = (long long)cdiv(N, G) * nbh * nbw * p.ncb;
        const double cost = (double)((nit + 256 * res - 1) / (256 * res)) * (busy > alone ? busy : alone);
        if (best.ok && cost >= best_cost) continue;
        p.ngrp = cdiv(N, G);
        const long long nitem = (long long)p.ngrp * nbh * nbw;
        if (nitem > (1 << 24)) continue;
        p.nitem = (int)nitem;
        best_cost = cost;
        best.p = p;
        best.S = S;
        best.lds_bytes = lds;
        best.ok = true;
      }
    }
  if (!best.ok) return best;
  Params& p = best.p;
  // items per workgroup: the fewest rounds of resident workgroups, each
  // costing its items and about one item of set-up
  const long long slots =
      256LL * resident(best.lds_bytes, waves, teams == 4 ? 2 : (op == kWgrad || op == kBwd ? 3 : 4));
  double span0 = -1.0;
  // at most 512 partial rows, and of the plain calls' at most kMaxPartBytes:
  // a size must not be too large for the fixed scratch only because it walks
  // (340 x 4142 x 39 x 39, K = 55: 9.1 MB, 0.9 MB with the table kernels)
  int rows = 512;
  if (op >= kWgrad && layout == kNCHW && str == 1 && mode == 0) {
    const long long fit = kMaxPartBytes / ((long long)C * K * 4);
    if (fit < rows) rows = fit < 1 ? 1 : (int)fit;
  }
  const int lo = cdiv(p.nitem, rows);
  for (int n = lo; n <= p.nitem; n += n < 64 ? 1 : n / 32) {
    const long long grid = (long long)p.ncb * cdiv(p.nitem, n);
    const double span = (double)((grid + slots - 1) / slots) * (n + 1.0);
    if (span0 < 0 || span <= span0) {
      span0 = span;
      p.ipw = n;
    }
  }
  p.runs = cdiv(p.nitem, p.ipw);
  const long long blocks = (long long)p.runs * p.ncb;
  if (blocks > 0x7fffffffll) {
    best.ok = false;
    return best;
  }
  p.nblocks = (int)blocks;
  p.xcd_per = p.nblocks % 8 == 0 ? p.nblocks / 8 : 0;
  best.parts = (size_t)p.runs;
  return best;
}

// Estimated times of a call with the walk and with the table-driven general
// kernels, in microseconds.  The table kernels: workgroups of `block` each,
// per pass the staged pixels and the cells times outputs of a lane, in whole
// rounds of resident workgroups or shared out over the CUs.  The walks:
// instructions per wave and item (cycles of the terms below), alone with their
// latencies or as many as share a SIMD, and a set-up per workgroup.  The rates
// are least-squares fits of the logarithms of 43477 pairs of timings (16000
// drawn calls: planes 7 .. 224 along a side, K 3 .. 63, every layout, stride
// 1 .. 3 and sampling, both storage types); on 16263 further ones the ratio of
// the two estimates has a standard deviation of 0.15 (small NHWC gathers) to
// 0.28 (NHWC weight gradients) in the logarithm.
struct Rates {
  double block, cell, cell16, fold, share, base;                            // table kernels (us; cell16: bfloat16's factor)
  double slot, slot16, store, step, phase, wait, piece, busy, setup, zero;  // walks (cycles; the last two us)
};
constexpr double kStageUs = 0.001;  // table kernels: a staged pixel
constexpr Rates kRates[3][2] = {  // [NCHW, NHWC, NHWC small][gathers, sums]
    {{1.63, 0.0103, 1.12, 0, 0.509, 6.04, 13.6, 0.903, 22.3, 17.8, 363, 20, 0, 1.89, 13.5, 2.61},
     {14.5, 0.0123, 1.42, 0, 0.405, 0.753, 28.2, 0.987, 12.1, 27.6, 466, 8.99, 2670, 1.32, 28.7, 2.79}},
    {{5.63, 0.0087, 1.37, 0, 0.724, 5.68, 18.3, 1.45, 137, 13.2, 251, 31, 3810, 1.3, 13.4, 0},
     {13.8, 0.0155, 1.7, 2.53, 0.664, 2.75, 18.8, 1.11, 95.3, 8.57, 161, 47, 4030, 1.3, 23.9, 0}},
    {{1.82, 0.0127, 1.21, 0, 0.785, 6.86, 16.7, 1.34, 75.3, 5.43, 168, 34, 0, 1.3, 7.44, 16.1},
     {2.88, 0.0349, 1.21, 0.789, 0.859, 10.1, 16.9, 1.17, 66.4, 5.85, 218, 29, 0, 1.3, 12.5, 20.7}}};
inline const Rates& rates_of(const Plan& pl, int op, int layout) {
  return kRates[layout == kNCHW ? 0 : (pl.p.small ? 2 : 1)][op >= kWgrad];
}

inline double table_us(const gen::Plan& pl, const Rates& r, int op, int layout, int esize) {
  const gen::Params& p = pl.p;
  const bool sums = op >= kWgrad;
  auto held = [&](int tile, int src) { return (double)(tile < (src - 1) * p.dil + 1 ? tile : (src - 1) * p.dil + 1) / p.dil; };
  const double staged = p.G * p.CB * held(p.TR, p.SH) * held(p.TC, p.SW);
  // a lane's tasks per pass; NHWC sums take up to four channels at a time
  const int cpp = p.CB < 4 ? p.CB : 4, wpc = 4 / cpp, npass = p.CB / cpp;
  const int tasks = layout == kNHWC && sums ? npass * cdiv(p.G * p.NRG * p.BQ, 64 * wpc)
                                            : cdiv(p.G * p.CB * p.NRG * p.BQ, gen::kThreads);
  const double cells = (double)tasks * p.ncap * p.RP * (sums ? p.nck : 1) * (esize == 2 ? r.cell16 : 1.0);
  const double folds = npass > 1 && sums ? r.fold * npass * p.nck : 0.0;
  const double block = r.block + (double)p.npw / p.G * (kStageUs * staged + r.cell * cells + folds);
  const int by_regs = !sums ? 8 : (p.KB <= 32 ? 4 : (p.KB <= 64 ? 3 : 2));
  const int by_lds = (int)((kMaxLdsBytes - 512) / ((pl.lds_bytes + 1023) / 1024 * 1024));
  const int slots = 256 * (by_lds < 1 ? 1 : (by_lds < by_regs ? by_lds : by_regs));
  const double shared = r.share * p.nblocks / 256 * block, rounds = (double)((p.nblocks + slots - 1) / slots) * block;
  return r.base + (shared > rounds ? shared : rounds);
}

inline double walk_us(const Plan& pl, const Rates& r, int op, int layout, int esize) {
  const Params& p = pl.p;
  const bool sums = op >= kWgrad;
  const int teams = layout == kNHWC ? 4 : 1, waves = teams * (p.small ? 64 : 128) / 64;
  const int res = resident(pl.lds_bytes, waves, teams == 4 ? 2 : (sums ? 3 : 4));
  const Staging sg = staging_of(p, layout, waves);
  const double instr = p.nph * (sg.slots * r.slot * (esize == 2 ? r.slot16 : 1.0) + r.phase) + p.K * (p.mode ? 2.4 : 1.0) * r.step +
                       cdiv(p.G * p.BH * p.BW, waves * 64) * r.store * (op == kDgrad ? p.nph : 1);
  const double alone = r.wait * instr + p.nph * r.piece * sg.pieces, busy = r.busy * instr * waves * res;
  const double block = p.ipw * (alone > busy ? alone : busy) / 2400.0 +
                       (r.setup + r.zero * (double)pl.lds_bytes / 65536.0) / 2.4;
  const double share = p.nblocks / (256.0 * res);
  const double rounds = 0.5 * ((p.nblocks + 256 * res - 1) / (256 * res) + (share > 1.0 ? share : 1.0));
  return 4.0 + rounds * block;
}

// Where the walks run instead of the table-driven general kernels: where they
// are large enough for the estimates above to count (`possible`: a walk pays
// about 5 us to build its program, more latency per staged phase, and for idle
// lanes of its 28-row strips), and the estimate is below 0.85 of the table
// kernels'.  Of 17724 timed calls that `possible` admits, 2801 were more than
// 5% slower walked (12 x 247 x 175 x 15, K = 21, NHWC: 117 against 96 us; 49 x
// 509 x 10 x 35, K = 9, bilinear, stride 2, NHWC: 410 against 63; 10 x 499 x
// 200 x 9, K = 33, bilinear: 566 against 175); of the 12574 that the estimate
// leaves, 334 are, and all calls together take 1.5% less time.
// `fill`: share of a team's lanes x rows that hold outputs.
inline bool possible(const Plan& pl, int op, int layout) {
  const Params& p = pl.p;
  const bool sums = op >= kWgrad;
  const double out = (double)p.N * p.C * p.P * p.Q;
  const double work = out * p.K * (p.mode ? 2.4 : 1.0) * 1e-6;  // million products
  const double fill = (double)p.G * p.BH * p.BW / (p.small ? 64.0 * kSmall : 128.0 * 28.0);
  if (p.str > 1) {
    // phases: small outputs wait for every phase's loads (2 x 64 x 56 x 56,
    // K = 17: 34 against 11 us); NHWC gains where the taps weigh (8 x 32 x
    // 112 x 112, K = 47: 40 against 79 us), NCHW on large planes (8 x 96 x
    // 224 x 224, K = 31: weight gradient 147 against 235 us), but not the
    // input gradient, whose phases stage dy again and store every other pixel
    if (layout == kNHWC) return work >= 25.0;
    return op != kDgrad && out >= 2e6 && p.P >= 64 && p.Q >= 64 && (sums || p.K <= 33);
  }
  if (layout == kNHWC) {
    // 32 x 128 x 7 x 7: K = 17 13 against 8 us, K = 47 13 against 17; 16 x 64 x
    // 30 x 30: K = 17 17 against 14, K = 47 23 against 27; 2 x 64 x 56 x 56,
    // K = 5: 16 against 20
    if (p.small) return work >= (sums ? 5.0 : 8.0);
    if (fill >= 0.5) return out >= 3e5;
    return fill >= (sums ? 0.12 : 0.22) && work >= (sums ? 10.0 : 40.0);
  }
  if (p.mode) {
    // bilinear, 2 x 64 x 56 x 56: K = 17 21 against 19 us, K = 47 28 against
    // 37; 16 x 64 x 30 x 30, K = 47, weight gradient 40 against 99
    if (fill >= 0.5) return work >= (sums ? 8.0 : 20.0);
    return work >= (sums ? 25.0 : 150.0);
  }
  // planes whose width the strip kernels do not take: 8 x 361 x 55 x 55, K = 15
  // both gradients 43 against 75 us; 32 x 80 x 45 x 37, K = 15 both gradients 43
  // against 47; 2 x 32 x 57 x 57, K = 15 15 against 10
  if (out < 2e6) return false;
  return sums ? fill >= 0.4 : fill >= 0.55 && work >= 20.0;
}

inline bool applies(const Plan& pl, const gen::Plan& table, int op, int layout, int esize) {
  if (!pl.ok || !possible(pl, op, layout)) return false;
  const Rates& r = rates_of(pl, op, layout);
  return !table.ok || walk_us(pl, r, op, layout, esize) < 0.85 * table_us(table, r, op, layout, esize);
}

}  // namespace walk

// Per storage type and layout; see o1d_walk_kernels.h.
#define O1D_WALK_DECL(T)                                                                                           \
  hipError_t launch_walk_gather_##T(const walk::Plan& pl, const void* in, const void* w, const float* theta,       \
                                    void* out, hipStream_t stream);                                                \
  hipError_t launch_walk_wgrad_##T(const walk::Plan& pl, const void* x, const void* dy, const float* theta,        \
                                   float* partial, hipStream_t stream);
O1D_WALK_DECL(f32_nchw)
O1D_WALK_DECL(f32_nhwc)
O1D_WALK_DECL(bf16_nchw)
O1D_WALK_DECL(bf16_nhwc)
#undef O1D_WALK_DECL
#define O1D_WALK_BDECL(T)                                                                                          \
  hipError_t launch_walk_bwd_##T(const walk::Plan& pl, const void* x, const void* dy, const void* w,               \
                                 const float* theta, void* dx, float* partial, hipStream_t stream);
O1D_WALK_BDECL(f32)
O1D_WALK_BDECL(bf16)
#undef O1D_WALK_BDECL

inline hipError_t launch_walk_gather(Dtype dt, const walk::Plan& pl, int layout, const void* in, const void* w,
                                     const float* theta, void* out, hipStream_t stream) {
  if (dt == Dtype::F32)
    return layout == walk::kNHWC ? launch_walk_gather_f32_nhwc(pl, in, w, theta, out, stream)
                                 : launch_walk_gather_f32_nchw(pl, in, w, theta, out, stream);
  return layout == walk::kNHWC ? launch_walk_gather_bf16_nhwc(pl, in, w, theta, out, stream)
                               : launch_walk_gather_bf16_nchw(pl, in, w, theta, out, stream);
}

inline hipError_t launch_walk_wgrad(Dtype dt, const walk::Plan& pl, int layout, const void* x, const void* dy,
                                    const float* theta, void* dw, float* partial, hipStream_t stream) {
  hipError_t e;
  if (dt == Dtype::F32)
    e = layout == walk::kNHWC ? launch_walk_wgrad_f32_nhwc(pl, x, dy, theta, partial, stream)
                              : launch_walk_wgrad_f32_nchw(pl, x, dy, theta, partial, stream);
  else
    e = layout == walk::kNHWC ? launch_walk_wgrad_bf16_nhwc(pl, x, dy, theta, partial, stream)
                              : launch_walk_wgrad_bf16_nchw(pl, x, dy, theta, partial, stream);
  return e != hipSuccess ? e : launch_partial_sum(dt, partial, dw, pl.p.C * pl.p.K, (int)pl.parts, stream);
}

inline hipError_t launch_walk_bwd(Dtype dt, const walk::Plan& pl, const void* x, const void* dy, const void* w,
                                  const float* theta, void* dx, void* dw, float* partial, hipStream_t stream) {
  const hipError_t e = dt == Dtype::F32 ? launch_walk_bwd_f32(pl, x, dy, w, theta, dx, partial, stream)
                                        : launch_walk_bwd_bf16(pl, x, dy, w, theta, dx, partial, stream);
  return e != hipSuccess ? e : launch_partial_sum(dt, partial, dw, pl.p.C * pl.p.K, (int)pl.parts, stream);
}

}  // namespace o1d
