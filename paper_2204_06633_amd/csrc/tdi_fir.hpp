// Kernels of the TDI filters (fir_tables.hpp): forward and transpose of one
// template, transpose of a batch, and the tables of the batched forward.
#pragma once

#include "batch_adjoint_kernels.hpp"
#include "fir_tables.hpp"

namespace lr {

// ---------------------------------------------------------------------------
// X, Y, Z (and A, E, T) of a tile of outputs per workgroup
// ---------------------------------------------------------------------------
template <int N, int GEN>
__global__ __launch_bounds__(kBlock, 4) void tdi_fir_kernel(TdiArgs a) {
  extern __shared__ double lds_dyn[];
  __shared__ FirShared sh;
  const int tid = threadIdx.x, K = a.fir_k, lo = a.fir_lo, half = (kFwdTile + K) / 2;
  double* W = lds_dyn + 12 * half;
  const int64_t i0 = xcd_tile(blockIdx.x, gridDim.x) * kFwdTile;
  const int cnt = (int)min((int64_t)kFwdTile, a.n_out - i0);
  const int64_t base = a.out_start + i0 + lo, ymax = a.n_y - 1;
  FirLane f;
  f.term = fir_lane_term<GEN>();
  bool bad = false;
  for (int k = tid; k < cnt + K; k += kBlock) {
    int64_t j = base + k;
    j = j < 0 ? 0 : (j > ymax ? ymax : j);
    double* d = lds_dyn + (k & 1) * half + (k >> 1);
#pragma unroll
    for (int l = 0; l < 6; ++l) {
      const double v = a.y[(int64_t)l * a.n_y + j];
      bad |= !(fabs(v) <= DBL_MAX);
      d[2 * half * l] = v;
    }
  }
  bad = __syncthreads_or(bad);

  const FirPiece P(0, cnt);
  const double t0 = a.t_off + (double)(a.out_start + i0) * a.dt;
  const bool one =
      fir_regular<GEN>(a.orb, t0 + P.c * a.dt, P.hw * a.dt, a.inv_dt, sh, f, W, 48 * K, tid);
  if (!one) fir_breaks<GEN>(a.orb, t0, a.dt, a.inv_dt, cnt, sh, tid);
#pragma unroll 1
  for (int p0 = 0; p0 < cnt;) {
    // an opaque lane index per piece: what derives from it is computed here
    // and not hoisted out of the loop into scratch
    int t = tid;
    asm volatile("" : "+v"(t));
    int len = cnt;
    if (!one) {
      len = fir_next(sh, p0, cnt) - p0;
      fir_shift(a.orb, t0 + (double)p0 * a.dt, a.inv_dt, sh, f, W, 48 * K, t);
    }
    fir_build<N, GEN, false>(f, lo, K, 0.0, W, t, bad);
    double v[2][3];
    if (!bad) {
      double S[3][2][4];
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) S[c][0][i] = S[c][1][i] = 0.0;
      const double* ev = lds_dyn + t;
      const double* od = ev + half;
      const double* w = W + (t & 15);
      static_for<6>([&](auto L) {
        constexpr int l = decltype(L)::value;
        constexpr int c0 = FirTab<GEN>::v.chan[2 * l], c1 = FirTab<GEN>::v.chan[2 * l + 1];
        // the next taps are read while these are summed; the last read ahead
        // stays inside the workgroup's LDS and is not used
        double y0 = ev[0], y1 = od[0], y2 = ev[1], x = w[0];
#pragma unroll 1
        for (int k = 1; k <= K / 2; ++k) {
          const double z1 = od[k], z2 = ev[k + 1], v = w[16 * k];
          fir_taps(S[c0], S[c1], x, y0, y1, y2);
          y0 = y2;
          y1 = z1;
          y2 = z2;
          x = v;
        }
        ev += 2 * half;
        od += 2 * half;
        w += 8 * K;
      });
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const double x = ((double)(2 * t + s) - P.c) * P.inv();
#pragma unroll
        for (int c = 0; c < 3; ++c) v[s][c] = fir_cubic(S[c][s], x);
      }
    } else {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const double x = ((double)(2 * t + s) - P.c) * P.inv();
#pragma unroll
        for (int c = 0; c < 3; ++c) v[s][c] = 0.0;
#pragma unroll 1
        for (int r = 0; r < 12; ++r) {
          const int c = fir_table<GEN>().chan[r];
          const double* w = W + (r >> 1) * 8 * K + (r & 1) * 4;
          const double* y = lds_dyn + 2 * half * (r >> 1) + t;
          double z = 0.0;
#pragma unroll 1
          for (int k = 0; k < K; ++k)
            z = fir_careful(w + 8 * k, x, y[((k + s) & 1) * half + ((k + s) >> 1)], z);
#pragma unroll
          for (int q = 0; q < 3; ++q) v[s][q] += q == c ? z : 0.0;
        }
      }
    }
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (2 * t + s >= p0 && 2 * t + s < p0 + len)
        store_channels(v[s], a.channels, a.out, a.n_out, i0 + 2 * t + s);
    p0 += len;
  }
}

template <int N, int GEN>
hipError_t launch_tdi_fir(const TdiArgs& a, hipStream_t s) {
  const int64_t blocks = (a.n_out + kFwdTile - 1) / kFwdTile;
  hipLaunchKernelGGL((tdi_fir_kernel<N, GEN>), dim3((unsigned)blocks), dim3(kBlock),
                     fir_lds_doubles(6, a.fir_k) * sizeof(double), s, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The transpose: g_y of a tile of link samples per workgroup, for M templates that
// share the filters.  Link sample s collects output s - out_start - lo - k
// over tap k; every element of g_y is written once (a tile in pieces adds
// the later pieces to what it wrote).
// ---------------------------------------------------------------------------
template <int N, int GEN, int M>
__device__ __forceinline__ void tdi_fir_adjoint_tile(const TdiAdjArgs (&a)[M],
                                                     const bool (&live)[M], int64_t tile,
                                                     double* lds, FirShared& sh) {
  const int tid = threadIdx.x, K = a[0].fir_k, lo = a[0].fir_lo, half = (kFwdTile + K) / 2;
  double* W = lds + 6 * M * half;
  const int64_t s0 = tile * kFwdTile;
  const int64_t ob = s0 - a[0].out_start - lo - (K - 1);     // output of window element 0
  int64_t n_out = a[0].n_out;
#pragma unroll
  for (int m = 1; m < M; ++m)
    if (live[m]) n_out = max(n_out, a[m].n_out);
  const int64_t o1 = max((int64_t)0, ob), o2 = min(n_out, ob + kFwdTile + K - 1);
  FirLane f;
  f.term = fir_lane_term<GEN>();
  if (o2 <= o1) {                                            // no output reaches the tile
#pragma unroll
    for (int m = 0; m < M; ++m)
      for (int i = tid; i < kFwdTile && live[m] && s0 + i < a[m].n_y; i += kBlock)
#pragma unroll
        for (int l = 0; l < 6; ++l) a[m].g_y[(int64_t)l * a[m].n_y + s0 + i] = 0.0;
    return;
  }
  const int n = (int)(o2 - o1);
  const FirPiece P(o1, n);
  const double dt = a[0].dt, inv_dt = a[0].inv_dt;
  const double t0 = a[0].t_off + (double)a[0].out_start * dt;        // time of output 0
  const bool one =
      fir_regular<GEN>(a[0].orb, t0 + P.c * dt, P.hw * dt, inv_dt, sh, f, W, 48 * K, tid);
  if (!one) fir_breaks<GEN>(a[0].orb, t0 + (double)o1 * dt, dt, inv_dt, n, sh, tid);
#pragma unroll 1
  for (int64_t p0 = o1; p0 < o2;) {
    int t = tid;
    asm volatile("" : "+v"(t));
    int len = n;
    if (!one) {
      len = fir_next(sh, (int)(p0 - o1), n) - (int)(p0 - o1);
      fir_shift(a[0].orb, t0 + (double)p0 * dt, inv_dt, sh, f, W, 48 * K, t);
    }
    // the piece's outputs, zero outside it
    bool bad = false;
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int64_t end = live[m] ? min(p0 + len, a[m].n_out) : p0;
      for (int k = t; k < kFwdTile + K; k += kBlock) {
        const int64_t o = ob + k;
        double g[3] = {0.0, 0.0, 0.0};
        if (o >= p0 && o < end) load_channel_grads(a[m].g_out, a[m].channels, a[m].n_out, o, g);
        double* d = lds + 6 * half * m + (k & 1) * half + (k >> 1);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          bad |= !(fabs(g[c]) <= DBL_MAX);
          d[2 * half * c] = g[c];
        }
      }
    }
    bad = __syncthreads_or(bad);
    fir_build<N, GEN, true>(f, lo, K, P.inv(), W, t, bad);
    const double x0 = ((double)(s0 + 2 * t - a[0].out_start) - P.c) * P.inv();
    const double x1 = ((double)(s0 + 2 * t + 1 - a[0].out_start) - P.c) * P.inv();
#pragma unroll 1
    for (int l = 0; l < 6; ++l) {
      const int c0 = fir_table<GEN>().chan[2 * l], c1 = fir_table<GEN>().chan[2 * l + 1];
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const double* eg = lds + 2 * half * (3 * m + c0) + t;
        const double* eh = lds + 2 * half * (3 * m + c1) + t;
        double v[2] = {0.0, 0.0};
        if (!bad) {
          const double* w = W + 8 * K * l + (t & 15);
          double S[2][4];
#pragma unroll
          for (int i = 0; i < 4; ++i) S[0][i] = S[1][i] = 0.0;
          double g0 = eg[0], g1 = eg[half], g2 = eg[1], h0 = eh[0], h1 = eh[half], h2 = eh[1];
          double x = w[0];
#pragma unroll 1
          for (int k = 1; k <= K / 2; ++k) {
            const double q1 = eg[half + k], q2 = eg[k + 1], r1 = eh[half + k], r2 = eh[k + 1];
            const double u = w[16 * k];
            fir_taps_adjoint(S, x, g0, g1, g2, h0, h1, h2);
            g0 = g2; g1 = q1; g2 = q2;
            h0 = h2; h1 = r1; h2 = r2;
            x = u;
          }
          v[0] = fir_cubic(S[0], x0);
          v[1] = fir_cubic(S[1], x1);
        } else {
#pragma unroll 1
          for (int k = 0; k < K; ++k) {
            const double* w = W + 8 * (K * l + k);
            const int a0 = (k & 1) * half + (k >> 1), a1 = ((k + 1) & 1) * half + ((k + 1) >> 1);
            v[0] = fir_careful(w, x0, eg[a0], v[0]);
            v[1] = fir_careful(w, x1, eg[a1], v[1]);
            v[0] = fir_careful(w + 4, x0, eh[a0], v[0]);
            v[1] = fir_careful(w + 4, x1, eh[a1], v[1]);
          }
        }
        double* dst = a[m].g_y + (int64_t)l * a[m].n_y + s0 + 2 * t;
#pragma unroll
        for (int s = 0; s < 2; ++s)
          if (live[m] && s0 + 2 * t + s < a[m].n_y) dst[s] = p0 == o1 ? v[s] : dst[s] + v[s];
      }
    }
    p0 += len;
  }
}

template <int N, int GEN>
__global__ __launch_bounds__(kBlock, 4) void tdi_fir_adjoint_kernel(TdiAdjArgs a) {
  extern __shared__ double lds_dyn[];
  __shared__ FirShared sh;
  const TdiAdjArgs x[1] = {a};
  const bool live[1] = {true};
  tdi_fir_adjoint_tile<N, GEN, 1>(x, live, xcd_tile(blockIdx.x, gridDim.x), lds_dyn, sh);
}

template <int N, int GEN>
hipError_t launch_tdi_fir_adjoint(const TdiAdjArgs& a, hipStream_t s) {
  const int64_t blocks = (a.n_y + kFwdTile - 1) / kFwdTile;
  hipLaunchKernelGGL((tdi_fir_adjoint_kernel<N, GEN>), dim3((unsigned)blocks), dim3(kBlock),
                     fir_lds_doubles(3, a.fir_k) * sizeof(double), s, a);
  return hipGetLastError();
}

// Batches: a pair of templates (sorted by duration) per work item shares the
// tables; every tile of the longer one's link samples is an item.  Measured on
// 12 templates of up to 788,941 outputs with the projection adjoint after it:
// 2.54 -> 1.81 ms, against the pairs of scatters that shared weight sequences.
template <int N, int GEN>
__global__ __launch_bounds__(kBlock, 4) void batch_tdi_fir_adjoint_kernel(BatchAdjArgs a) {
  extern __shared__ double lds_dyn[];
  __shared__ FirShared sh;
  const int64_t item = xcd_tile(blockIdx.x, gridDim.x);
  const int64_t pr = a.items[2 * item], tile = a.items[2 * item + 1];
  const int64_t b0 = a.pairs[2 * pr], b1 = a.pairs[2 * pr + 1];
  TdiAdjArgs x[2] = {batch_tdi_args(a, a.tpl[b0]), batch_tdi_args(a, a.tpl[b1 >= 0 ? b1 : b0])};
  x[0].fir_lo = x[1].fir_lo = a.fir_lo;
  x[0].fir_k = x[1].fir_k = a.fir_k;
  const bool live[2] = {true, b1 >= 0 && tile * kFwdTile < x[1].n_y};
  tdi_fir_adjoint_tile<N, GEN, 2>(x, live, tile, lds_dyn, sh);
}

template <int N, int GEN>
hipError_t launch_batch_tdi_fir_adjoint(const BatchAdjArgs& a, int64_t n_items, hipStream_t s) {
  const size_t bytes = fir_lds_doubles(6, a.fir_k) * sizeof(double);
  hipLaunchKernelGGL((batch_tdi_fir_adjoint_kernel<N, GEN>), dim3((unsigned)n_items), dim3(kBlock),
                     bytes, s, a);
  return hipGetLastError();
}

// Tables of the batched forward: one workgroup per interval of kFirInterval
// outputs, built in LDS and stored; a flag where a delay crosses an integer within
// the interval.  The workgroups after them do what precedes a fused
// forward anyway (run_forward_prep): the work counter and the sky angles'
// sines and cosines.
template <int N, int GEN>
__global__ __launch_bounds__(kBlock, 4) void fir_tables_kernel(BatchFwdArgs a) {
  extern __shared__ double lds_dyn[];
  __shared__ FirShared sh;
  const int tid = threadIdx.x, K = a.fir_k;
  const int64_t q = blockIdx.x;
  if (q >= a.n_fir) {
    const int64_t k = (q - a.n_fir) * kBlock + tid;
    if (k == 0) *a.counter = 0;
    if (k < a.n_templates) {
      double sn, cs;
      sincos(a.sky[a.sky_stride * k], &sn, &cs);
      a.trig[4 * k] = sn;
      a.trig[4 * k + 1] = cs;
      sincos(a.sky[a.sky_stride * k + 1], &sn, &cs);
      a.trig[4 * k + 2] = sn;
      a.trig[4 * k + 3] = cs;
    }
    return;
  }
  FirLane f;
  f.term = fir_lane_term<GEN>();
  const FirPiece P(q * kFirInterval, kFirInterval);
  const bool ok = fir_regular<GEN>(a.orb_t, a.t_off_t + P.c * a.dt, P.hw * a.dt, a.inv_dt, sh, f,
                                   lds_dyn, 48 * K, tid);
  fir_build<N, GEN, false>(f, a.fir_lo, K, 0.0, lds_dyn, tid, true);
  // four taps of a link as 16 pairs, so that a lane loads them at once
  const int nq = fir_quads(K), n = 192 * nq;
  double* w = a.fir + q * n;
  for (int e = tid; e < n; e += kBlock) {
    const int l = e / (32 * nq), r = e - l * 32 * nq, p = 2 * (r >> 5) + (r & 1);
    w[e] = 2 * p < K ? lds_dyn[l * 8 * K + 16 * p + ((r >> 1) & 15)] : 0.0;
  }
  if (tid == 0) a.fir_split[q] = !ok;
}

template <int N, int GEN>
hipError_t launch_fir_tables(const BatchFwdArgs& a, hipStream_t s) {
  const int64_t blocks = a.n_fir + (a.n_templates + kBlock - 1) / kBlock;
  hipLaunchKernelGGL((fir_tables_kernel<N, GEN>), dim3((unsigned)blocks), dim3(kBlock),
                     (size_t)48 * a.fir_k * sizeof(double), s, a);
  return hipGetLastError();
}

#define LR_INSTANTIATE_FIR(NT)                                                       \
  template hipError_t launch_tdi_fir<NT, 1>(const TdiArgs&, hipStream_t);            \
  template hipError_t launch_tdi_fir<NT, 2>(const TdiArgs&, hipStream_t);            \
  template hipError_t launch_tdi_fir_adjoint<NT, 1>(const TdiAdjArgs&, hipStream_t); \
  template hipError_t launch_tdi_fir_adjoint<NT, 2>(const TdiAdjArgs&, hipStream_t); \
  template hipError_t launch_batch_tdi_fir_adjoint<NT, 1>(const BatchAdjArgs&, int64_t, \
                                                          hipStream_t);              \
  template hipError_t launch_batch_tdi_fir_adjoint<NT, 2>(const BatchAdjArgs&, int64_t, \
                                                          hipStream_t); \
  template hipError_t launch_fir_tables<NT, 1>(const BatchFwdArgs&, hipStream_t);    \
  template hipError_t launch_fir_tables<NT, 2>(const BatchFwdArgs&, hipStream_t);

}  // namespace lr
