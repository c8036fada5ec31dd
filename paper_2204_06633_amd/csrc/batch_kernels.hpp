// Batched response kernels for gfx950 (FP64): many templates (sources or
// MCMC walkers) sharing one output time grid, one launch.
//
// fused_forward_kernel<N, GEN, M, BLOCK, WAVE> is persistent: each workgroup
// takes work items (a group of M templates, a tile of output samples) from an
// atomic counter until the list is exhausted.  For one item it
//   1. computes, template by template, the link series of the tile plus the
//      TDI halo directly into LDS (projection, Sec. IV.B, farrow_forward.hpp)
//      -- the link series never reaches HBM;
//   2. evaluates TDI (Sec. IV.C) for all M templates at once: the delays
//      depend on the orbits only, so each filter weight (fir_tables.hpp), or
//      each Lagrange coefficient sequence in an interval that no filter serves,
//      is formed once per sample and applied to the M templates' series;
//   3. stores X/Y/Z and/or A/E/T of each template.
// Batches without filters (fused_fir_shape) run stream_forward_kernel instead.
#pragma once

#include "batch_stream_kernels.hpp"
#include "farrow_forward.hpp"
#include "fir_tables.hpp"

namespace lr {

// TDI of the lane's two outputs for M templates from the filters: W the lane's position in its interval's table
// (its DPP row's 16 coefficients), j0 the row element of its first output's
// first tap, t, u powers of the two outputs' times in the interval.  A weight
// is computed once and applied to the M templates: 12 K (4 + M) / M
// instructions per output and template.
template <int GEN, int M, int YR>
__device__ __forceinline__ void fused_tdi_fir(const double* ylds, const double2* W, int K, int j0,
                                              const double (&t)[3], const double (&u)[3],
                                              double (&acc)[M][2][3]) {
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[m][0][c] = acc[m][1][c] = 0.0;
  const int NQ = fir_quads(K);
  // elements j0 + k for even and odd k
  const double* ev = ylds + par<YR>(j0);
  const double* od = ylds + par<YR>(j0 + 1);
  static_for<6>([&](auto L) {
    constexpr int l = decltype(L)::value;
    constexpr int c0 = FirTab<GEN>::v.chan[2 * l], c1 = FirTab<GEN>::v.chan[2 * l + 1];
    double y0[M], y1[M];
    double2 w = W[0];
#pragma unroll
    for (int m = 0; m < M; ++m) {
      y0[m] = ev[m * 6 * YR];
      y1[m] = od[m * 6 * YR];
    }
    auto pair = [&](double x, int k) {
      // the link samples of the next taps are read while these are summed
      double y2[M], z1[M];
      const int kz = min(k + 1, K / 2 - 1);
#pragma unroll
      for (int m = 0; m < M; ++m) {
        y2[m] = ev[m * 6 * YR + k + 1];
        z1[m] = od[m * 6 * YR + kz];
      }
      double p[2], r[2];
      fir_weights<0>(x, t, u, p, r);
#pragma unroll
      for (int m = 0; m < M; ++m) {
        acc[m][0][c0] = fma(p[0], y0[m], acc[m][0][c0]);
        acc[m][1][c0] = fma(p[1], y1[m], acc[m][1][c0]);
        acc[m][0][c1] = fma(r[0], y0[m], acc[m][0][c1]);
        acc[m][1][c1] = fma(r[1], y1[m], acc[m][1][c1]);
      }
      fir_weights<1>(x, t, u, p, r);
#pragma unroll
      for (int m = 0; m < M; ++m) {
        acc[m][0][c0] = fma(p[0], y1[m], acc[m][0][c0]);
        acc[m][1][c0] = fma(p[1], y2[m], acc[m][1][c0]);
        acc[m][0][c1] = fma(r[0], y1[m], acc[m][0][c1]);
        acc[m][1][c1] = fma(r[1], y2[m], acc[m][1][c1]);
        y0[m] = y2[m];
        y1[m] = z1[m];
      }
    };
#pragma unroll 1
    for (int q = 0; q < NQ; ++q) {
      const double2 v = W[16 * min(q + 1, NQ - 1)];     // four taps ahead
      pair(w.x, 2 * q);
      if (2 * q + 1 < K / 2) pair(w.y, 2 * q + 1);
      w = v;
    }
    W += 16 * NQ;
    ev += YR;
    od += YR;
  });
}

// The same with the same bits where link samples of the segment are not finite: a tap
// that is empty must not spread a NaN or an infinity past the stencils, and is passed
// over.  tab: the interval's table.
template <int GEN, int M, int YR>
__device__ __forceinline__ void fused_tdi_careful(const double* ylds, const double* tab, int K,
                                                  int j0, const double (&t)[3],
                                                  const double (&u)[3], double (&acc)[M][2][3]) {
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[m][0][c] = acc[m][1][c] = 0.0;
#pragma unroll 1
  for (int l = 0; l < 6; ++l)
#pragma unroll 1
    for (int k = 0; k < K; ++k)
#pragma unroll 1
      for (int i = 0; i < 2; ++i) {
        const int ch = fir_table<GEN>().chan[2 * l + i];
        const double* w = tab + 32 * (l * fir_quads(K) + (k >> 2)) + ((k >> 1) & 1) +
                          16 * (k & 1) + 8 * i;
        const double c0 = w[0], c1 = w[2], c2 = w[4], c3 = w[6];
        if (c0 == 0.0 && c1 == 0.0 && c2 == 0.0 && c3 == 0.0) continue;
        const double p = fma(c3, t[2], fma(c2, t[1], fma(c1, t[0], c0)));
        const double r = fma(c3, u[2], fma(c2, u[1], fma(c1, u[0], c0)));
#pragma unroll
        for (int m = 0; m < M; ++m) {
          const double* y = ylds + (m * 6 + l) * YR;
          const double a = y[par<YR>(j0 + k)], b = y[par<YR>(j0 + k + 1)];
#pragma unroll
          for (int c = 0; c < 3; ++c)
            if (c == ch) {
              acc[m][0][c] = fma(p, a, acc[m][0][c]);
              acc[m][1][c] = fma(r, b, acc[m][1][c]);
            }
        }
      }
}

// WAVE: h+ / hx synthesised from each template's parameter row (Sec. III)
// instead of read from the caller's arrays.  A compile-time choice: with the
// waveform code in the same kernel the array path's registers spill.  Two waves per
// SIMD: LDS lets no more workgroups of the usual shapes share a CU, and the
// projection's coefficients need the registers.
template <int N, int GEN, int M, int BLOCK, bool WAVE>
__global__ __launch_bounds__(BLOCK, 2)
void fused_forward_kernel(BatchFwdArgs a) {
  constexpr int HPX = fused_halo_cap(M, BLOCK);       // halo a row can carry
  constexpr int YR = kPerLane * BLOCK + HPX;          // row length
  constexpr int NST = (M * 6 * HPX + BLOCK - 1) / BLOCK;   // halo values per lane (<= 2)
  static_assert(NST <= 2, "two halo values per lane");
  __shared__ __align__(16) double ylds[M * 6 * YR];
  __shared__ FarrowForward<N, BLOCK, 5, 32> proj;
  __shared__ int s_item;
  const int YT = a.samples;                           // new link samples per tile

  for (;;) {
    // an opaque lane index per item: whatever derives from it (LDS offsets,
    // stencil starts) is recomputed here instead of being hoisted out of the
    // persistent loop and kept in scratch
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    if (tid == 0) s_item = atomicAdd(a.counter, 1);
    __syncthreads();
    // uniform values in scalar registers: the item, its group and segment,
    // and (below) the templates' records come through scalar loads
    const int item = __builtin_amdgcn_readfirstlane(s_item);
    if (item >= a.n_items) break;
    const int grp = __builtin_amdgcn_readfirstlane(a.items[2 * item]);
    const int seg = __builtin_amdgcn_readfirstlane(a.items[2 * item + 1]);
    const int hp = a.HP;                              // 0: one tile per segment
    const int64_t S = (int64_t)seg * (a.T_out + (int64_t)(a.seg_tiles - 1) * YT);
    const int64_t n_long = a.tpl[grp * M].n_out;      // the group's longest template
    // A segment is seg_tiles consecutive tiles.  Row r of a tile holds link
    // sample rb + r (output-index space, rb = first output - F - ro): the
    // tile's new link samples go to rows [hp, hp + YT); from the second
    // tile on, rows [0, hp) hold the previous tile's last hp samples, so
    // every tile after the first has YT outputs.
    double halo[NST > 0 ? NST : 1];
    bool bad = false;                                 // a link sample of the segment is not finite
#pragma unroll 1
    for (int t = 0; t < a.seg_tiles; ++t) {
      const int64_t o0 = t == 0 ? S : S + a.T_out + (int64_t)(t - 1) * YT;
      if (o0 >= n_long) break;                        // uniform
      const int cnt = t == 0 ? a.T_out : YT;          // outputs of this tile
      const int ro = t == 0 ? hp : 0;
      const int64_t i_new = o0 - a.F + (t == 0 ? 0 : hp);   // link sample of row hp

      // 1. link series of each template of the group into LDS (one copy of the
      // projection code, templates in a rolled loop)
      bool live[M];
#pragma unroll
      for (int k = 0; k < M; ++k) {
        const BatchTemplate T = a.tpl[grp * M + k];
        live[k] = T.index >= 0 && o0 < T.n_out;
      }
#pragma unroll 1
      for (int k = 0; k < M; ++k) {
        const BatchTemplate T = a.tpl[grp * M + k];
        if (!(T.index >= 0 && o0 < T.n_out)) continue;  // uniform
        const int64_t n_valid = min((int64_t)cnt, T.n_out - o0);
        // new rows up to the last valid output's stencil (the padding B
        // rounded to the even halo YT - T_out)
        const int r_end =
            (int)min((int64_t)YT, n_valid + a.halo - (t == 0 ? 0 : hp));
        // sin, cos of the sky angles, tabulated per template before the launch
        // (no trigonometry, and none of its constants, in this loop)
        const double* tr = a.trig + 4 * T.index;
        const Sky sk = sky_from_trig(tr[0], tr[1], tr[2], tr[3]);
        // h+ / hx: the caller's arrays, or the waveform synthesised into the
        // window from the template's parameter row (waveform time 0 at output
        // sample 0)
        HSource hs;
        if constexpr (WAVE)
          hs = HSource::waveform(a.params + 8 * T.index, -T.out_start, a.dt, T.n_h);
        else
          hs = HSource::arrays(a.hp + T.h_off, a.hc + T.h_off, T.n_h);
#pragma unroll 1
        for (int r0 = 0; r0 < r_end; r0 += a.rows) {
          const int n = min(a.rows, r_end - r0);
          double y[6];
          proj.project(a.orb_p, a.t_off_p, i_new + r0, a.dt, a.inv_dt, hs,
                       T.out_start + i_new + r0, sk, tid, n, y);
          if (tid < n) {
#pragma unroll
            for (int l = 0; l < 6; ++l) {
              ylds[(k * 6 + l) * YR + par<YR>(hp + r0 + tid)] = y[l];
              bad |= !(fabs(y[l]) <= DBL_MAX);
            }
          }
        }
        if (t > 0) {
          // the carried halo of this template back into its rows
#pragma unroll
          for (int q = 0; q < NST; ++q) {
            const int e = tid + BLOCK * q, rho = e / max(HPX, 1), j = e - rho * HPX;
            if (rho / 6 == k && rho < M * 6 && j < hp) ylds[rho * YR + par<YR>(j)] = halo[q];
          }
        }
      }
      // 2. TDI of the tile's outputs for all live templates
      // tile-relative output of sample a; a row of 16 lanes starts at a multiple
      // of 32 outputs, so that it lies in one interval of the filters
      const int oa = 2 * tid - (int)(o0 & 31);
      const bool out_a = oa >= 0 && oa < cnt;
      const int ob = max(0, min(oa, cnt - 2));        // idle lanes mirror the ends
      double acc[M][2][3];
      bad = __syncthreads_or(bad);
      bool split = false;
      {
        // outputs past the longest template of the batch have no interval, and
        // are not stored
        const int64_t o = o0 + ob;
        const int qe = (int)a.n_fir - 1, q = min((int)(o / kFirInterval), qe);
        const int q0 = (int)(o0 / kFirInterval), q1 = min((int)((o0 + cnt - 1) / kFirInterval), qe);
        const double c = (double)q * kFirInterval + 0.5 * (kFirInterval - 1);
        constexpr double inv = 2.0 / (kFirInterval - 1);
        double ta[3], tb[3];
        ta[0] = ((double)o - c) * inv;
        tb[0] = ((double)(o + 1) - c) * inv;
        ta[1] = ta[0] * ta[0];
        tb[1] = tb[0] * tb[0];
        ta[2] = ta[1] * ta[0];
        tb[2] = tb[1] * tb[0];
        const double2* W = reinterpret_cast<const double2*>(a.fir) +
                           (int64_t)q * 96 * fir_quads(a.fir_k);
        const int j0 = a.F + a.fir_lo + ro + ob;
        if (!bad)
          fused_tdi_fir<GEN, M, YR>(ylds, W + (tid & 15), a.fir_k, j0, ta, tb, acc);
        else
          fused_tdi_careful<GEN, M, YR>(ylds, &W->x, a.fir_k, j0, ta, tb, acc);
        for (int i = q0; i <= q1; ++i) split |= a.fir_split[i] != 0;
      }
      if (split) {                                    // uniform
        double La[6], Lb[6], one[M][2][3];
        light_times(a.orb_t, a.t_off_t + (double)(o0 + ob) * a.dt, La);
        light_times(a.orb_t, a.t_off_t + (double)(o0 + ob + 1) * a.dt, Lb);
        fused_tdi<N, GEN, M, YR, false>(a, ylds, La, Lb, a.F + ro + ob, live, one);
        const bool mine = a.fir_split[min((o0 + ob) / kFirInterval, a.n_fir - 1)] != 0;
#pragma unroll
        for (int k = 0; k < M; ++k)
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int c = 0; c < 3; ++c) acc[k][s][c] = mine ? one[k][s][c] : acc[k][s][c];
      }

      // 3. store (the template records read again rather than kept live
      // through the TDI: an opaque copy of the group index stops the compiler
      // from reusing the first loads)
      int grp_s = grp;
      asm volatile("" : "+s"(grp_s));
      if (out_a) {
#pragma unroll
        for (int k = 0; k < M; ++k) {
          if (!live[k]) continue;
          const BatchTemplate T = a.tpl[grp_s * M + k];
          const int64_t i = o0 + oa;
          if (i < T.n_out) store_channels(acc[k][0], a.channels, a.out + T.out_off, T.n_out, i);
          if (i + 1 < T.n_out)
            store_channels(acc[k][1], a.channels, a.out + T.out_off, T.n_out, i + 1);
        }
      }
      if (t + 1 < a.seg_tiles) {
        // the next tile's halo: this tile's last hp link samples, read before
        // the next tile's projection windows overwrite them
        const int from = t == 0 ? hp + a.T_out : YT;
#pragma unroll
        for (int q = 0; q < NST; ++q) {
          const int e = tid + BLOCK * q, rho = e / max(HPX, 1), j = e - rho * HPX;
          if (rho < M * 6 && j < hp) halo[q] = ylds[rho * YR + par<YR>(from + j)];
        }
      }
      __syncthreads();                                // LDS free for the next tile
    }
  }
}

template <int N, int GEN, int M, int BLOCK, bool WAVE>
hipError_t launch_fused_forward(const BatchFwdArgs& a, int blocks, hipStream_t s) {
  if (a.fir_k > 0)
    hipLaunchKernelGGL((fused_forward_kernel<N, GEN, M, BLOCK, WAVE>), dim3(blocks), dim3(BLOCK),
                       0, s, a);
  else
    hipLaunchKernelGGL((stream_forward_kernel<N, GEN, M, BLOCK, WAVE>), dim3(blocks), dim3(BLOCK),
                       0, s, a);
  return hipGetLastError();
}

// Resident workgroups per CU (sizes the persistent grid), of the roomier of the
// two kernels: a workgroup that starts late finds the work list drained.
template <int N, int GEN, int M, int BLOCK, bool WAVE>
int fused_occupancy() {
  int f = 0, t = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &f, fused_forward_kernel<N, GEN, M, BLOCK, WAVE>, BLOCK, 0) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &t, stream_forward_kernel<N, GEN, M, BLOCK, WAVE>, BLOCK, 0) != hipSuccess)
    return 1;
  return f > t ? (f > 0 ? f : 1) : (t > 0 ? t : 1);
}

#define LR_INSTANTIATE_BATCH_FWD_M(NT, GEN, M, BLOCK, WAVE)                              \
  template hipError_t launch_fused_forward<NT, GEN, M, BLOCK, WAVE>(const BatchFwdArgs&, int, \
                                                                    hipStream_t);             \
  template int fused_occupancy<NT, GEN, M, BLOCK, WAVE>();

// Work items of 256, 512 or 1024 link samples (workgroups of 128, 256 or 512
// lanes); groups of 4 at 1024 would need 196 KB of LDS and are left out.
// Waveform mode: groups of 1 and 2 at 512 link samples and of 2 at 1024 (the
// fastest array-mode shapes), which keeps the build time in bounds.
#define LR_INSTANTIATE_BATCH_FWD(NT, GEN)                                                   \
  LR_INSTANTIATE_BATCH_FWD_M(NT, GEN, 1, 128, false)                                        \
  LR_INSTANTIATE_BATCH_FWD_M(NT, GEN, 1, 256, false)                                        \
  LR_INSTANTIATE_BATCH_FWD_M(NT, GEN, 1, 512, false)                                        \
  LR_INSTANTIATE_BATCH_FWD_M(NT, GEN, 2, 128, false)                                        \
  LR_INSTANTIATE_BATCH_FWD_M(NT, GEN, 2, 256, false)                                        \
  LR_INSTANTIATE_BATCH_FWD_M(NT, GEN, 2, 512, false)                                        \
  LR_INSTANTIATE_BATCH_FWD_M(NT, GEN, 4, 128, false)                                        \
  LR_INSTANTIATE_BATCH_FWD_M(NT, GEN, 4, 256, false)                                        \
  LR_INSTANTIATE_BATCH_FWD_M(NT, GEN, 1, 256, true)                                         \
  LR_INSTANTIATE_BATCH_FWD_M(NT, GEN, 2, 256, true)                                         \
  LR_INSTANTIATE_BATCH_FWD_M(NT, GEN, 2, 512, true)

}  // namespace lr
