// TDI and its transpose as short filters with slowly varying taps (FP64, gfx950).
//
// An output channel is a sum of delayed link terms (Sec. IV.C), each an
// N-tap Lagrange interpolation (Sec. IV.E).  The delays are chains of light
// times, which change by about 1e-7 of a sample per sample, so over a tile of
// 512 samples every interpolation weight is, to rounding, a cubic in time, and
// the 3 or 4 terms that one link contributes to one channel overlap: their
// weights add up to one filter of K = N - 1 + ceil(longest delay / dt) taps.
// A workgroup builds the twelve (link, channel) filters at four Chebyshev
// nodes of its tile, turns them into cubics, and then spends four FMAs per
// tap, filter and sample: 12 K x 4 = 1536 at order 25 and dt = 10 s, against
// 4524 for 36 weight sequences and 42 streams.  The filters do not depend on
// the template.  The same table transposed is the adjoint, as a gather: no
// atomics, no zero fill, and a fixed order of additions.
//
// Bound: FP64 vector issue.  One year at dt = 10 s, order 25, TDI-2 (3,155,760
// outputs): forward 0.535 -> 0.232 ms, of which about 0.16 ms are the filter
// FMAs (31 T/s of the 34 T/s a plain FMA loop reaches), 0.05 ms the tables and
// the rest loads and stores; transpose 0.842 -> 0.260 ms.  Tiles of 512 with
// 256 lanes: four workgroups share a CU and hide each other's table phase
// (1024 with 512 lanes halves the tables but measured 0.267 ms).
//
// The expansion is exact to rounding where the light times are smooth, which the
// host judges (fir_taps in api.cpp), and while every delay keeps its integer shift.
// A tile in which one crosses an integer finds the outputs where that happens and
// takes the pieces between them in turn, with the cubics of the whole tile: the
// shift changes from piece to piece, the fraction just runs past 0 or 1.  With
// Keplerian orbits few tiles of a year are such tiles (at most 2 in 100, where dt is
// near a light time), of two or three pieces; a template of 1400 outputs with 25 to
// 50 pieces in one tile (order 25, dt = 10 s) takes 190 to 300 us, and took up to
// 1600 where the pieces were found by bisection (25 in one piece).
#pragma once

#include <float.h>

#include "forward_kernels.hpp"

namespace lr {

// Terms of a filter row (row 2 l + i is the i-th channel that link l feeds),
// packed: 4 bits for each link light time's multiplicity in the delay, then
// bit 24: the term exists, bit 25: it is subtracted.  An undelayed term has
// all multiplicities zero.
constexpr uint32_t kFirTermBit = 1u << 24, kFirMinusBit = 1u << 25;

template <int GEN>
struct FirTable {
  static constexpr int kTerms = GEN == 1 ? 2 : 4;   // per row
  uint32_t term[12 * kTerms];                 // [term][row]
  int chan[12];
};

template <int GEN>
constexpr FirTable<GEN> make_fir_table() {
  constexpr TdiTable<GEN> t = make_tdi_table<GEN>();
  FirTable<GEN> r{};
  int fed[6][2] = {}, nfed[6] = {}, nt[12] = {};
  auto add = [&](const int (&cnt)[6], const GroupUse& u) {
    int i = 0;
    while (i < nfed[u.link] && fed[u.link][i] != u.chan) ++i;
    const int q = 2 * u.link + i;
    if (i == nfed[u.link]) {
      fed[u.link][nfed[u.link]++] = u.chan;
      r.chan[q] = u.chan;
    }
    uint32_t w = kFirTermBit | (u.sign < 0 ? kFirMinusBit : 0u);
    for (int l = 0; l < 6; ++l) w |= (uint32_t)cnt[l] << (4 * l);
    r.term[12 * nt[q]++ + q] = w;
  };
  constexpr int none[6] = {0, 0, 0, 0, 0, 0};
  for (int i = 0; i < t.ndirect; ++i)
    add(none, GroupUse{t.direct[i].chan, t.direct[i].sign, t.direct[i].link});
  for (int g = 0; g < t.ngroup; ++g)
    for (int u = 0; u < t.group[g].nuse; ++u) add(t.group[g].cnt, t.group[g].use[u]);
  return r;
}

template <int GEN>
struct FirTab {
  static constexpr FirTable<GEN> v = make_fir_table<GEN>();
};

static __constant__ FirTable<1> kFir1 = make_fir_table<1>();
static __constant__ FirTable<2> kFir2 = make_fir_table<2>();

template <int GEN>
__device__ __forceinline__ const FirTable<GEN>& fir_table() {
  if constexpr (GEN == 1) return kFir1;
  else return kFir2;
}

// Outputs per table of the batched forward, from output 0 of the batch: fixed,
// so that no result depends on how a batch is cut into tiles.
constexpr int kFirInterval = kFwdTile;

// Nodes of the cubic in time (Chebyshev), then the ends of the interval.
constexpr double kFirX0 = 0.92387953251128674, kFirX1 = 0.38268343236508977;

__device__ __forceinline__ double fir_point(int p) {
  const double v = p == 0 || p == 3 ? kFirX0 : p == 1 || p == 2 ? kFirX1 : 1.0;
  return p == 2 || p == 3 || p == 4 ? -v : v;
}

// Most outputs of an interval: a tile of the transpose is reached by kFwdTile + K - 1.
constexpr int kFirMost = kFwdTile + 128;

struct FirShared {
  double L[6][6];                      // light times at the six points
  unsigned long long brk[kFirMost / 64];   // outputs at which a delay's shift changes
};

// One term of one filter row at one node, held by lane 4 (12 term + row) +
// node of the workgroup.
struct FirLane {
  uint32_t term;
  double a, shift;     // -delay / dt at the lane's node, its integer part on the piece
};

template <int GEN>
__device__ __forceinline__ uint32_t fir_lane_term() {
  constexpr int n = 12 * FirTable<GEN>::kTerms;
  const int i = threadIdx.x >> 2;
  return i < n ? fir_table<GEN>().term[i] : 0u;
}

// Delay of a term whose link light times are L, in seconds.
__device__ __forceinline__ double fir_delay(uint32_t term, const double (&L)[6]) {
  double d = 0.0;
#pragma unroll
  for (int l = 0; l < 6; ++l) d = fma((double)((term >> (4 * l)) & 15u), L[l], d);
  return d;
}

// What rounding leaves open of a = -delay / dt: an excess over an integer of this
// size is let through (the fraction then leaves [0, 1] by that much, where the two
// stencils agree).
__device__ __forceinline__ double fir_tolerance(double a) { return 1e-15 - 1e-15 * a; }

// Light times of the interval (centre tc, half width hs seconds on the orbit
// grid), the lane's term on it, and whether every delay has one integer shift s
// (s <= a <= s + 1): judged at the nodes and the ends, the extent of a widened by
// a quarter of itself (the delay between the points).  Barriers inside; W (n
// doubles) is cleared on the way.
template <int GEN>
__device__ __forceinline__ bool fir_regular(const OrbitView& orb, double tc, double hs,
                                            double inv_dt, FirShared& sh, FirLane& f, double* W,
                                            int n, int tid) {
  // opaque copies: the term's decoding stays in here instead of being hoisted
  // out of the callers' loops into scratch
  uint32_t term = f.term;
  asm volatile("" : "+v"(tid), "+v"(term));
  __syncthreads();
  if (tid < 36) {
    const int p = tid / 6, l = tid - 6 * p;
    double u;
    const double* seg = orbit_segment(orb, tc + hs * fir_point(p), u);
    sh.L[p][l] = spline_at(seg, 9 + l, u);
  }
  for (int e = tid; e < n; e += kBlock) W[e] = 0.0;
  __syncthreads();
  const double a = -fir_delay(term, sh.L[tid & 3]) * inv_dt;
  const double b = -fir_delay(term, sh.L[4 + (tid & 1)]) * inv_dt;
  double lo = fmin(a, b), hi = fmax(a, b);
  lo = fmin(lo, __shfl_xor(lo, 1));
  hi = fmax(hi, __shfl_xor(hi, 1));
  lo = fmin(lo, __shfl_xor(lo, 2));
  hi = fmax(hi, __shfl_xor(hi, 2));
  const double change = hi - lo, tol = fir_tolerance(lo);
  f.a = a;
  f.shift = floor(lo - 0.25 * change + tol);
  return __syncthreads_and(hi + 0.25 * change - tol <= f.shift + 1.0);
}

// The outputs among n (the first at time t0 on the orbit grid) at which some
// delay's shift differs from the output before: every lane compares two
// neighbours, the shifts folded into one number in base 3 (a delay changes by far
// less than a sample over an interval, so a shift by one at most).
template <int GEN>
__device__ __forceinline__ void fir_breaks(const OrbitView& orb, double t0, double dt,
                                           double inv_dt, int n, FirShared& sh, int tid) {
  const GroupTable<GEN>& GT = group_table<GEN>();
  auto fold = [&](int o) {
    double u, L[6];
    const double* seg = orbit_segment(orb, t0 + (double)o * dt, u);
#pragma unroll
    for (int l = 0; l < 6; ++l) L[l] = spline_at(seg, 9 + l, u);
    unsigned long long h = 0;
#pragma unroll 1
    for (int g = 0; g < GT.n; ++g) {
      const double a = -row_delay(GT.row[g], L) * inv_dt;
      h = 3 * h + (unsigned long long)(long long)floor(a + fir_tolerance(a));
    }
    return h;
  };
#pragma unroll 1
  for (int o = tid; o < kFirMost; o += kBlock) {
    const bool at = o > 0 && o < n && fold(o) != fold(o - 1);
    const unsigned long long m = __ballot(at);
    if ((tid & 63) == 0) sh.brk[o >> 6] = m;
  }
  __syncthreads();
}

// First output after p at which a shift changes, or n.
__device__ __forceinline__ int fir_next(const FirShared& sh, int p, int n) {
  int w = (p + 1) >> 6;
  unsigned long long m = w < kFirMost / 64 ? sh.brk[w] & (~0ull << ((p + 1) & 63)) : 0;
  while (m == 0 && ++w < kFirMost / 64) m = sh.brk[w];
  return m ? min(n, 64 * w + (int)__ffsll(m) - 1) : n;
}

// The lane's shift on the piece that starts at time t0.  Barriers inside; W is
// cleared on the way.
__device__ __forceinline__ void fir_shift(const OrbitView& orb, double t0, double inv_dt,
                                          FirShared& sh, FirLane& f, double* W, int n, int tid) {
  __syncthreads();
  if (tid < 6) {
    double u;
    const double* seg = orbit_segment(orb, t0, u);
    sh.L[4][tid] = spline_at(seg, 9 + tid, u);
  }
  for (int e = tid; e < n; e += kBlock) W[e] = 0.0;
  __syncthreads();
  const double a = -fir_delay(f.term, sh.L[4]) * inv_dt;
  f.shift = floor(a + fir_tolerance(a));
}

// The filters of the interval as cubics in the interval's own time t in
// [-1, 1], to the cleared W[link][k][row of the link][4] (K taps, tap k at
// link sample o + lo + k of output o).  mark: a weight that is exactly zero (a delay
// of whole samples) leaves its tap in the stencil, though a trace only, so that a
// NaN there still counts.  TRANS: for the transpose, taps in
// reverse order, and the cubics moved to the link sample's time (output =
// link sample - lo - k; inv_hw: 1 / half width in samples).
template <int N, int GEN, bool TRANS>
__device__ __forceinline__ void fir_build(const FirLane& f, int lo, int K, double inv_hw,
                                          double* W, int tid, bool mark) {
  const int rq = tid >> 2, r = rq % 12, q = rq / 12;
  const bool direct = (f.term & 0xffffffu) == 0;
  const double sign = f.term & kFirMinusBit ? -1.0 : 1.0;
  double w[N];
  lagrange_weights<N>(f.a - f.shift, w, sign);
  if (mark) {
#pragma unroll
    for (int m = 0; m < N; ++m) w[m] = w[m] == 0.0 ? 1e-300 : w[m];
  }
  const int kb = min(max((int)f.shift - (N / 2 - 1) - lo, 0), K - N);
  double* row = W + (r >> 1) * 8 * K + (r & 1) * 4 + (tid & 3);
  // the terms of a row are added in turn
#pragma unroll 1
  for (int t = 0; t < FirTable<GEN>::kTerms; ++t) {
    if (q == t && (f.term & kFirTermBit)) {
      if (direct) {
        row[8 * -lo] += sign;
      } else {
        // reads in blocks ahead of the writes, which may alias them
        double* at = row + 8 * kb;
        constexpr int B = 6;
#pragma unroll
        for (int m = 0; m < N; m += B) {
          double v[B];
#pragma unroll
          for (int i = 0; i < B; ++i)
            if (m + i < N) v[i] = at[8 * (m + i)];
#pragma unroll
          for (int i = 0; i < B; ++i)
            if (m + i < N) at[8 * (m + i)] = v[i] + w[m + i];
        }
      }
    }
    __syncthreads();
  }
  // node values -> coefficients
  auto coef = [&](const double* v, int k, double (&c)[4]) {
    const double e0 = 0.5 * (v[0] + v[3]), e1 = 0.5 * (v[1] + v[2]);
    const double o0 = (v[0] - v[3]) * (0.5 / kFirX0), o1 = (v[1] - v[2]) * (0.5 / kFirX1);
    constexpr double X = 1.0 / (kFirX0 * kFirX0 - kFirX1 * kFirX1);
    c[2] = (e0 - e1) * X;
    c[3] = (o0 - o1) * X;
    c[0] = fma(-kFirX0 * kFirX0, c[2], e0);
    c[1] = fma(-kFirX0 * kFirX0, c[3], o0);
    if constexpr (TRANS) {
      const double x = -(double)(lo + k) * inv_hw;
      c[0] = fma(x, fma(x, fma(x, c[3], c[2]), c[1]), c[0]);
      c[1] = fma(x, fma(3.0 * x, c[3], 2.0 * c[2]), c[1]);
      c[2] = fma(3.0 * x, c[3], c[2]);
    }
  };
  auto put = [](double* d, const double (&c)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = c[i];
  };
  if constexpr (!TRANS) {
    for (int e = tid; e < 12 * K; e += kBlock) {
      double c[4];
      coef(W + 4 * e, 0, c);
      put(W + 4 * e, c);
    }
  } else {
    for (int e = tid; e < 6 * K; e += kBlock) {
      const int l = e / K, k = (e - l * K) >> 1, i = e & 1;   // k < K / 2
      double* a = W + l * 8 * K + k * 8 + i * 4;
      double* b = W + l * 8 * K + (K - 1 - k) * 8 + i * 4;
      double ca[4], cb[4];
      coef(a, k, ca);
      coef(b, K - 1 - k, cb);
      put(a, cb);
      put(b, ca);
    }
  }
  __syncthreads();
}

// Two taps of one link for both samples of a lane: p, q are the sums of the
// link's two channels by power of the time, w holds the 16 coefficients of
// the taps in the 16 lanes of every DPP row, y0, y1, y2 the link samples of
// tap k (sample a), of k + 1 (a) and k (b), and of k + 1 (b).  The broadcast
// rides on the FMA (row_newbcast), so a weight costs no scalar register, no
// LDS broadcast and no extra instruction; the s_nop covers the wait states of
// a DPP operand, which the compiler does not see here.
__device__ __forceinline__ void fir_taps(double (&p)[2][4], double (&q)[2][4], double w, double y0,
                                         double y1, double y2) {
  asm(
      "s_nop 1\n"
      "v_fmac_f64_dpp %0, %16, %17 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %4, %16, %18 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %16, %17 row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %5, %16, %18 row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %16, %17 row_newbcast:2 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %6, %16, %18 row_newbcast:2 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %16, %17 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %7, %16, %18 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %8, %16, %17 row_newbcast:4 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %12, %16, %18 row_newbcast:4 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %9, %16, %17 row_newbcast:5 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %13, %16, %18 row_newbcast:5 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %10, %16, %17 row_newbcast:6 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %14, %16, %18 row_newbcast:6 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %11, %16, %17 row_newbcast:7 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %15, %16, %18 row_newbcast:7 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %16, %18 row_newbcast:8 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %4, %16, %19 row_newbcast:8 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %16, %18 row_newbcast:9 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %5, %16, %19 row_newbcast:9 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %16, %18 row_newbcast:10 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %6, %16, %19 row_newbcast:10 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %16, %18 row_newbcast:11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %7, %16, %19 row_newbcast:11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %8, %16, %18 row_newbcast:12 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %12, %16, %19 row_newbcast:12 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %9, %16, %18 row_newbcast:13 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %13, %16, %19 row_newbcast:13 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %10, %16, %18 row_newbcast:14 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %14, %16, %19 row_newbcast:14 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %11, %16, %18 row_newbcast:15 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %15, %16, %19 row_newbcast:15 row_mask:0xf bank_mask:0xf\n"
      : "+v"(p[0][0]), "+v"(p[0][1]), "+v"(p[0][2]), "+v"(p[0][3]), "+v"(p[1][0]), "+v"(p[1][1]),
        "+v"(p[1][2]), "+v"(p[1][3]), "+v"(q[0][0]), "+v"(q[0][1]), "+v"(q[0][2]), "+v"(q[0][3]),
        "+v"(q[1][0]), "+v"(q[1][1]), "+v"(q[1][2]), "+v"(q[1][3])
      : "v"(w), "v"(y0), "v"(y1), "v"(y2));
}

// The transpose: one link, two inputs (the gradients g, h of its two
// channels).
__device__ __forceinline__ void fir_taps_adjoint(double (&p)[2][4], double w, double g0, double g1,
                                                 double g2, double h0, double h1, double h2) {
  asm(
      "s_nop 1\n"
      "v_fmac_f64_dpp %0, %8, %9 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %4, %8, %10 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %8, %9 row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %5, %8, %10 row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %8, %9 row_newbcast:2 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %6, %8, %10 row_newbcast:2 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %8, %9 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %7, %8, %10 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %8, %12 row_newbcast:4 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %4, %8, %13 row_newbcast:4 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %8, %12 row_newbcast:5 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %5, %8, %13 row_newbcast:5 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %8, %12 row_newbcast:6 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %6, %8, %13 row_newbcast:6 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %8, %12 row_newbcast:7 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %7, %8, %13 row_newbcast:7 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %8, %10 row_newbcast:8 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %4, %8, %11 row_newbcast:8 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %8, %10 row_newbcast:9 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %5, %8, %11 row_newbcast:9 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %8, %10 row_newbcast:10 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %6, %8, %11 row_newbcast:10 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %8, %10 row_newbcast:11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %7, %8, %11 row_newbcast:11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %8, %13 row_newbcast:12 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %4, %8, %14 row_newbcast:12 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %8, %13 row_newbcast:13 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %5, %8, %14 row_newbcast:13 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %8, %13 row_newbcast:14 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %6, %8, %14 row_newbcast:14 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %8, %13 row_newbcast:15 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %7, %8, %14 row_newbcast:15 row_mask:0xf bank_mask:0xf\n"
      : "+v"(p[0][0]), "+v"(p[0][1]), "+v"(p[0][2]), "+v"(p[0][3]), "+v"(p[1][0]), "+v"(p[1][1]),
        "+v"(p[1][2]), "+v"(p[1][3])
      : "v"(w), "v"(g0), "v"(g1), "v"(g2), "v"(h0), "v"(h1), "v"(h2));
}

// The weights of tap TAP (0 or 1) of a pair for two samples a, b of a lane (t, u:
// first to third power of their times): c0, c1 the link's two channels.  Used
// where several templates share a weight: four instructions for it, then one
// FMA per template.
template <int TAP>
__device__ __forceinline__ void fir_weights(double w, const double (&t)[3], const double (&u)[3],
                                            double (&c0)[2], double (&c1)[2]) {
  if constexpr (TAP == 0)
    asm("s_nop 1\n"
      "v_mov_b64_dpp %0, %4 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"
      "v_mov_b64_dpp %1, %4 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"
      "v_mov_b64_dpp %2, %4 row_newbcast:4 row_mask:0xf bank_mask:0xf\n"
      "v_mov_b64_dpp %3, %4 row_newbcast:4 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %4, %5 row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %4, %6 row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %4, %5 row_newbcast:5 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %4, %6 row_newbcast:5 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %4, %7 row_newbcast:2 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %4, %8 row_newbcast:2 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %4, %7 row_newbcast:6 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %4, %8 row_newbcast:6 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %4, %9 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %4, %10 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %4, %9 row_newbcast:7 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %4, %10 row_newbcast:7 row_mask:0xf bank_mask:0xf\n"
        : "=&v"(c0[0]), "=&v"(c0[1]), "=&v"(c1[0]), "=&v"(c1[1])
        : "v"(w), "v"(t[0]), "v"(u[0]), "v"(t[1]), "v"(u[1]), "v"(t[2]), "v"(u[2]));
  else
    asm("s_nop 1\n"
      "v_mov_b64_dpp %0, %4 row_newbcast:8 row_mask:0xf bank_mask:0xf\n"
      "v_mov_b64_dpp %1, %4 row_newbcast:8 row_mask:0xf bank_mask:0xf\n"
      "v_mov_b64_dpp %2, %4 row_newbcast:12 row_mask:0xf bank_mask:0xf\n"
      "v_mov_b64_dpp %3, %4 row_newbcast:12 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %4, %5 row_newbcast:9 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %4, %6 row_newbcast:9 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %4, %5 row_newbcast:13 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %4, %6 row_newbcast:13 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %4, %7 row_newbcast:10 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %4, %8 row_newbcast:10 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %4, %7 row_newbcast:14 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %4, %8 row_newbcast:14 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %4, %9 row_newbcast:11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %4, %10 row_newbcast:11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %4, %9 row_newbcast:15 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %4, %10 row_newbcast:15 row_mask:0xf bank_mask:0xf\n"
        : "=&v"(c0[0]), "=&v"(c0[1]), "=&v"(c1[0]), "=&v"(c1[1])
        : "v"(w), "v"(t[0]), "v"(u[0]), "v"(t[1]), "v"(u[1]), "v"(t[2]), "v"(u[2]));
}

__device__ __forceinline__ double fir_cubic(const double (&c)[4], double t) {
  return fma(t, fma(t, fma(t, c[3], c[2]), c[1]), c[0]);
}

// x + w y where the tap is not empty: an empty tap must not spread a NaN or an
// infinity of the series beyond the stencils.
__device__ __forceinline__ double fir_careful(const double* w, double t, double y, double x) {
  const double c[4] = {w[0], w[1], w[2], w[3]};
  const bool empty = c[0] == 0.0 && c[1] == 0.0 && c[2] == 0.0 && c[3] == 0.0;
  return empty ? x : fma(fir_cubic(c, t), y, x);
}

// LDS doubles of the kernels: rows of a tile + K samples split by parity
// (a lane reads element 2 lane + k: consecutive addresses across the wave),
// then the filters.
__host__ __device__ constexpr size_t fir_lds_doubles(int rows, int K) {
  return (size_t)rows * (kFwdTile + K) + 48 * K + 16;   // + 16: read ahead
}

// An interval of len outputs from output p0 on as centre (samples) and half width.
struct FirPiece {
  double c, hw;
  __device__ __forceinline__ FirPiece(int64_t p0, int64_t len)
      : c((double)p0 + 0.5 * (double)(len - 1)), hw(0.5 * (double)(len - 1)) {}
  __device__ __forceinline__ double inv() const { return hw > 0.0 ? 1.0 / hw : 0.0; }
};

}  // namespace lr
