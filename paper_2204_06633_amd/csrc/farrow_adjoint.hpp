// Projection adjoint and sky gradient in one pass (FP64, gfx950): the
// transpose of the nine interpolations per link sample, and the gradient with
// respect to the sky angles, from polynomials per stencil base (farrow.hpp).
//
// A workgroup of 256 lanes takes two runs of `rows` consecutive link samples,
// rows = 256 minus the spread of the nine positions, so that 256 stencil bases
// cover a run.  Per run:
//   A. lane = link sample: geometry, u and integer part of each position, and
//      the gradient of each position's h+ and hx, to LDS;
//   B. lane = stencil base J: coefficients of h+ and hx, then position by
//      position the link sample r = J - shift it serves: value and derivative
//      for the sky angles back into r's LDS slots, and the gradients times
//      powers of u added to J's coefficient gradients; at the end these turn
//      into the gradients of the N samples around J, summed in the wave's own
//      LDS row (LDS adds of one wave stay in order), then over the waves, and
//      added to the zero-filled gradients.  An element receives at most two
//      additions there, so results are bitwise reproducible -- but for positions
//      further apart than `rows` allows for, which are served one after the other,
//      and for ones that move so fast that runs are halved: then more meet.
//   C. lane = link sample: sky gradient from the values and derivatives.
//
// Bound by FP64 issue at two waves per SIMD (registers: 64 coefficients and
// coefficient gradients per lane).  One year at dt = 10 s, order 25, against
// nine weight sequences per link sample: with the sky gradient 804 -> 441 us,
// without 380 -> 245 us (order 1: 191 -> 150; order 13: 272 -> 209).  With
// predicates and a list of steps in phase B throughout, as where integer parts
// cross within a run, it took 541 and 306 us where this took 506 and 245.
#pragma once

#include "batch_adjoint_kernels.hpp"
#include "farrow.hpp"

namespace lr {

// Rows of the LDS arrays: the quick path of phase B takes positions up to
// kFarrowPad apart, where a base's link sample is its lane minus up to that; what
// lies before a row's first link sample is zero.
constexpr int kFarrowPad = 16, kFarrowLd = kFarrowBlock + kFarrowPad;

// A step of phase B's general path: the link samples whose position `row` has
// integer part f; k = f minus the position's smallest.
struct FarrowStep {
  int row, f, k, end;
};
constexpr int kFarrowSteps = 48;               // most steps of a run

struct FarrowShared {
  int lo[kFarrowBlock / 64][9], hi[kFarrowBlock / 64][9];   // per wave: integer parts
  alignas(16) FarrowStep step[kFarrowSteps + 3];
  double s_trig[2][2];
  double s_part[9][kFarrowBlock / 64];         // per wave: sky gradient, waveform sums
  gb::Source src;
  unsigned char f[9 * kFarrowBlock];           // integer part minus lo
};

// Doubles of dynamic LDS: u and the two gradients per position and link
// sample, the window of h+ and hx (wave: and of the phase's sine and cosine,
// which the parameter sums use again: eight templates of a million samples 1.74
// -> 1.71 ms), and the waves' sums.
__host__ __device__ constexpr size_t farrow_adjoint_doubles(int N, bool window, bool wave) {
  return 27 * kFarrowLd + ((window ? 2 : 0) + (wave ? 2 : 0)) * (kFarrowBlock + N) +
         (kFarrowBlock / 64) * 2 * (64 + N);
}

template <int N, bool SKY, bool WAVE>
__device__ __forceinline__ void farrow_adjoint_tile(const ProjAdjArgs& a, int64_t tile,
                                                    double* lds, FarrowShared& sh,
                                                    double* part_out) {
  constexpr int H = N / 2, D = FarrowTable<N>::D, LD = kFarrowLd, WR = 64 + N;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  double* U = lds + kFarrowPad;
  double* GP = U + 9 * LD;
  double* GC = U + 18 * LD;
  double2* win = reinterpret_cast<double2*>(lds + 27 * LD);
  static_assert(SKY || !WAVE, "the window holds the waveform");
  double2* trigs = win + kFarrowBlock + N;
  double* sums = lds + 27 * LD + ((SKY ? 2 : 0) + (WAVE ? 2 : 0)) * (kFarrowBlock + N);
  double* mine = sums + wv * 2 * WR;

  load_sky(a.sky, sh.s_trig);
  // the sky basis from its trigonometry in LDS, where it is needed
  auto trig = [&]() {
    int i = 0;
    asm volatile("" : "+v"(i));
    const double* t = &sh.s_trig[0][0] + i;
    return SkyTrig{t[0], t[1], t[2], t[3]};
  };
  // h+ and hx: the arrays, or the waveform with its constants kept in LDS
  if (WAVE && tid == 0) sh.src = gb::load_source(a.params);
  if (lane < 9) sh.s_part[lane][wv] = 0.0;
  for (int e = tid; e < 27 * kFarrowPad; e += kFarrowBlock)
    U[e / kFarrowPad * LD - 1 - e % kFarrowPad] = 0.0;
  __syncthreads();
  auto source = [&]() {
    if constexpr (WAVE) {
      int i = 0;
      asm volatile("" : "+v"(i));
      return HSource::waveform((&sh.src)[i], a.k0, a.dt, a.n_h);
    } else {
      return HSource::arrays(a.hp, a.hc, a.n_h);
    }
  };
  // a lane's share of sum `slot`, added over the wave and to the wave's total
  auto add_up = [&](double v, int slot) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (lane == 0) sh.s_part[slot][wv] += v;
  };
  const int64_t end = min(a.n_y, (tile + 1) * kFarrowRuns * a.rows);
  int most = a.rows;
#pragma unroll 1
  for (int64_t r0 = tile * kFarrowRuns * a.rows; r0 < end;) {
    int n = (int)min((int64_t)most, end - r0);
    int t = tid;                               // opaque: nothing hoisted out of the loop
    asm volatile("" : "+v"(t));
    const int rel = min(t, n - 1);
    const bool active = t < n;
    const int64_t q0 = a.y_start + r0;
    const double tau = a.t_off + (double)(q0 + rel) * a.dt;

    // A.
    int f[9], wlo = 0;                         // lane p < 9: the range of position p
    {
      double gl[6];
#pragma unroll
      for (int l = 0; l < 6; ++l) {
        gl[l] = a.g_y[(int64_t)l * a.n_y + r0 + rel];
        gl[l] = active ? gl[l] : 0.0;
      }
      LinkGeom g;
      const SkyTrig tr = trig();
      link_geometry(a.orb, tau, sky_from_trig(tr.sl, tr.cl, tr.sb, tr.cb), g);
      double u[9];
      int differ = 0;
#pragma unroll
      for (int p = 0; p < 9; ++p) {
        f[p] = split_centred(position_delay(g, p), a.inv_dt, u[p]);
        const int f0 = __builtin_amdgcn_readfirstlane(f[p]);
        differ |= f[p] ^ f0;
        wlo = lane == p ? f0 : wlo;
      }
      int whi = wlo;
      if (__any(differ)) {
#pragma unroll
        for (int p = 0; p < 9; ++p) {
          const int x = wave_min(f[p]), y = wave_max(f[p]);
          wlo = lane == p ? x : wlo;
          whi = lane == p ? y : whi;
        }
      }
      if (lane < 9) {
        sh.lo[wv][lane] = wlo;
        sh.hi[wv][lane] = whi;
      }
#pragma unroll
      for (int l = 0; l < 6; ++l) gl[l] *= 0.5 * fast_rcp(1.0 - kDir[l] * g.kn[kArm[l]]);
      __syncthreads();                         // lo, hi; the previous run is done with LDS
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        double vp = 0.0, vc = 0.0;
#pragma unroll
        for (int l = 0; l < 6; ++l)
          if (kLinkRecv[l] - 1 == i) {
            vp = fma(-gl[l], g.xip[kArm[l]], vp);
            vc = fma(-gl[l], g.xic[kArm[l]], vc);
          }
        GP[i * LD + t] = vp;
        GC[i * LD + t] = vc;
      }
#pragma unroll
      for (int l = 0; l < 6; ++l) {
        GP[(3 + l) * LD + t] = gl[l] * g.xip[kArm[l]];
        GC[(3 + l) * LD + t] = gl[l] * g.xic[kArm[l]];
      }
#pragma unroll
      for (int p = 0; p < 9; ++p) U[p * LD + t] = u[p];
    }
    const int pl = min(lane, 8);
    int whi = sh.hi[0][pl];
    wlo = sh.lo[0][pl];
#pragma unroll
    for (int w = 1; w < kFarrowBlock / 64; ++w) {
      wlo = min(wlo, sh.lo[w][pl]);
      whi = max(whi, sh.hi[w][pl]);
    }
    int jlo = 1 << 30, jhi = -(1 << 30), drift = 0, steps = 0;
#pragma unroll
    for (int p = 0; p < 9; ++p) {
      const int x = __builtin_amdgcn_readlane(wlo, p), y = __builtin_amdgcn_readlane(whi, p);
      jlo = min(jlo, x);
      jhi = max(jhi, y);
      drift = max(drift, y - x);
      steps += y - x + 1;
    }
    // One set of bases for all positions when they lie as close together as
    // the light times say (the host's `rows`); else one per position, and
    // fewer link samples where the positions themselves move too fast.
    const bool together = n + jhi - jlo <= kFarrowBlock;
    const bool fast = together && drift == 0 && jhi - jlo <= kFarrowPad;
    if (n > 1 && (n + drift > kFarrowBlock || steps > kFarrowSteps)) {
      most = max(1, n / 2);
      __syncthreads();                         // lo, hi read before they are set again
      continue;
    }
    if (!fast) {
      int at = 0;
#pragma unroll
      for (int p = 0; p < 9; ++p) {
        const int x = __builtin_amdgcn_readlane(wlo, p), y = __builtin_amdgcn_readlane(whi, p);
        sh.f[p * kFarrowBlock + t] = (unsigned char)(f[p] - x);
        if (t == p)
          for (int i = 0; i <= y - x; ++i) sh.step[at + i] = FarrowStep{p, x + i, i, 0};
        at += y - x + 1;
      }
      if (t == 9)                              // the list's end, and what is read ahead of it
        sh.step[at] = sh.step[at + 1] = sh.step[at + 2] = FarrowStep{0, 0, 0, 1};
    }
    __syncthreads();                           // fractions, gradients, steps

    // B.
#pragma unroll 1
    for (int g = 0; g < (together ? 1 : 9); ++g) {
      int base = jlo, nj = n + jhi - jlo;
      if (!together) {
        base = __builtin_amdgcn_readlane(wlo, g);
        nj = n + __builtin_amdgcn_readlane(whi, g) - base;
      }
      const int64_t j0 = q0 + base - (H - 1);  // h-index of window element 0
      double cp[D + 1], cc[D + 1], dp[D + 1], dc[D + 1];
      if constexpr (SKY) {
        const HSource hs = source();
        for (int k = t; k < nj + N - 1; k += kFarrowBlock) {
          int64_t j = j0 + k;
          j = j < 0 ? 0 : (j > a.n_h - 1 ? a.n_h - 1 : j);
          if constexpr (WAVE)
            win[k] = hs.at(j, trigs[k]);
          else
            win[k] = hs.at(j);
        }
        __syncthreads();
        farrow_coefs<N>(win + min(t, nj - 1), cp, cc);
      }
#pragma unroll
      for (int m = 0; m <= D; ++m) dp[m] = dc[m] = 0.0;
      for (int e = lane; e < 2 * WR; e += 64) mine[e] = 0.0;
      // a position's share of the coefficient gradients, and with SKY its
      // values vp, vc and the derivative ds along its delay
      auto serve = [&](double u, double gp, double gc, double& vp, double& vc, double& ds) {
        if constexpr (SKY) {
          double wp = cp[D], wc = cc[D];       // derivatives
          vp = cp[D];
          vc = cc[D];
#pragma unroll
          for (int m = D - 1; m >= 0; --m) {
            vp = fma(vp, u, cp[m]);
            vc = fma(vc, u, cc[m]);
            if (m > 0) {
              wp = fma(wp, u, vp);
              wc = fma(wc, u, vc);
            }
          }
          ds = fma(gp, wp, gc * wc);
        }
        dp[0] += gp;
        dc[0] += gc;
        double pw = u;
#pragma unroll
        for (int m = 1; m <= D; ++m) {
          dp[m] = fma(gp, pw, dp[m]);
          dc[m] = fma(gc, pw, dc[m]);
          if (m < D) pw *= u;
        }
      };
      if (fast) {
        // base t serves link sample t + jlo - f of each position: before the
        // run's first and after its last the gradients are zero.  The next
        // position's LDS reads are issued before this one's sums.
        int at = t + jlo - __builtin_amdgcn_readlane(wlo, 0);
        double u = U[at], gp = GP[at], gc = GC[at];
#pragma unroll 1
        for (int p = 0; p < 9; ++p) {
          const int q = min(p + 1, 8);
          const int an = t + q * LD + jlo - __builtin_amdgcn_readlane(wlo, q);
          const double un = U[an], gpn = GP[an], gcn = GC[an];
          double vp, vc, ds;
          serve(u, gp, gc, vp, vc, ds);
          if constexpr (SKY) {
            if ((unsigned)(at - p * LD) < (unsigned)n) {
              U[at] = ds;
              GP[at] = vp;
              GC[at] = vc;
            }
          }
          at = an;
          u = un;
          gp = gpn;
          gc = gcn;
        }
      } else {
        // Step by step, each step's LDS reads issued before the previous
        // step's sums: the link sample r served by this base and its u and
        // gradients, zero where this base serves none.
        struct Item {
          int at;
          bool ok;
          double u, gp, gc;
        };
        auto fetch = [&](const FarrowStep& st) {
          Item it;
          const int r = t + base - st.f, rc = min(max(r, 0), n - 1);
          it.at = st.row * LD + rc;
          it.ok = r == rc && (int)sh.f[st.row * kFarrowBlock + rc] == st.k;
          it.u = U[it.at];
          it.gp = GP[it.at];
          it.gc = GC[it.at];
          return it;
        };
        auto uniform = [](const FarrowStep& v) {
          return FarrowStep{
              __builtin_amdgcn_readfirstlane(v.row), __builtin_amdgcn_readfirstlane(v.f),
              __builtin_amdgcn_readfirstlane(v.k), __builtin_amdgcn_readfirstlane(v.end)};
        };
        int i = 0;
        if (!together)
          while (__builtin_amdgcn_readfirstlane(sh.step[i].row) != g) ++i;
        Item it = fetch(uniform(sh.step[i]));
        FarrowStep nxt = uniform(sh.step[i + 1]), later = sh.step[i + 2];
        i += 2;
#pragma unroll 1
        for (;;) {
          const Item ahead = fetch(nxt);
          const bool last = nxt.end || (!together && nxt.row != g);
          nxt = uniform(later);
          later = sh.step[min(++i, kFarrowSteps + 2)];
          double vp, vc, ds;
          serve(it.ok ? it.u : 0.0, it.ok ? it.gp : 0.0, it.ok ? it.gc : 0.0, vp, vc, ds);
          if constexpr (SKY) {
            if (it.ok) {
              U[it.at] = ds;
              GP[it.at] = vp;
              GC[it.at] = vc;
            }
          }
          it = ahead;
          if (last) break;
        }
      }
      // coefficient gradients -> gradients of the samples j0 + t + k, added to
      // the wave's own sums tap after tap (LDS adds of one wave keep their
      // order)
      farrow_transpose<N>(dp, dc, [&](int k, double gp, double gc) {
        unsafeAtomicAdd(mine + lane + k, gp);
        unsafeAtomicAdd(mine + WR + lane + k, gc);
      });
      __syncthreads();
      double acc[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
      const HSource hs = source();
      for (int e = t; e < nj + N - 1; e += kFarrowBlock) {
        double v[2] = {0.0, 0.0};
#pragma unroll
        for (int w = 0; w < kFarrowBlock / 64; ++w) {
          const int i = e - 64 * w;
          if (i >= 0 && i < WR - 1) {
            v[0] += sums[w * 2 * WR + i];
            v[1] += sums[w * 2 * WR + WR + i];
          }
        }
        const int64_t j = j0 + e;
        if (j >= 0 && j < a.n_h) {
          if constexpr (WAVE) {
            // the lane that filled this element of the window
            const double2 sc = trigs[e];
            gb::adjoint_sums(hs.src, (double)(a.k0 + j) * a.dt, sc.x, sc.y, v[0], v[1], acc);
          } else {
            atomicAdd(a.g_hp + j, v[0]);
            atomicAdd(a.g_hc + j, v[1]);
          }
        }
      }
      if constexpr (WAVE) {
#pragma unroll
        for (int k = 0; k < 7; ++k) add_up(acc[k], 2 + k);
      }
      if (!together) __syncthreads();          // the next position's window and sums
    }

    // C.
    if constexpr (SKY) {
      const double inv_cdt = a.inv_dt / kC;
      LinkGeom g;
      const SkyTrig tr = trig();
      int rc = rel;
      asm volatile("" : "+v"(rc));             // read and computed again, not kept through B
      double gy[6];
#pragma unroll
      for (int l = 0; l < 6; ++l) gy[l] = a.g_y[(int64_t)l * a.n_y + r0 + rc];
      link_geometry(a.orb, a.t_off + (double)(q0 + rc) * a.dt,
                    sky_from_trig(tr.sl, tr.cl, tr.sb, tr.cb), g);
      // the derivatives along each spacecraft's delay
      double s[3], Gk[3], Gu[3] = {0.0, 0.0, 0.0}, Gv[3] = {0.0, 0.0, 0.0};
#pragma unroll
      for (int i = 0; i < 3; ++i) s[i] = U[i * LD + rel];
#pragma unroll
      for (int l = 0; l < 6; ++l) s[kLinkEmit[l] - 1] += U[(3 + l) * LD + rel];
#pragma unroll
      for (int c = 0; c < 3; ++c)
        Gk[c] = -inv_cdt * (s[0] * g.x[0][c] + s[1] * g.x[1][c] + s[2] * g.x[2][c]);
#pragma unroll
      for (int l = 0; l < 6; ++l) {
        const int arm = kArm[l], r = kLinkRecv[l] - 1;
        const double hp = GP[(3 + l) * LD + rel] - GP[r * LD + rel];
        const double hc = GC[(3 + l) * LD + rel] - GC[r * LD + rel];
        const double inv = fast_rcp(1.0 - kDir[l] * g.kn[arm]);
        const double gl = 0.5 * gy[l] * inv;
        const double sn = gl * inv * kDir[l] * (g.xip[arm] * hp + g.xic[arm] * hc);
        const double su = 2.0 * gl * (g.un[arm] * hp + g.vn[arm] * hc);
        const double sv = 2.0 * gl * (g.un[arm] * hc - g.vn[arm] * hp);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          Gk[c] = fma(sn, g.n[arm][c], Gk[c]);
          Gu[c] = fma(su, g.n[arm][c], Gu[c]);
          Gv[c] = fma(sv, g.n[arm][c], Gv[c]);
        }
      }
      const SkyDeriv sd = sky_derivatives(tr.sl, tr.cl, tr.sb, tr.cb);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        double v = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c)
          v += Gk[c] * sd.dk[i][c] + Gu[c] * sd.du[i][c] + Gv[c] * sd.dv[i][c];
        add_up(active ? v : 0.0, i);
      }
    }
    r0 += n;
  }

  // the waves' totals in wave order
  if constexpr (SKY || WAVE) {
    __syncthreads();
    if (tid < 9) {
      double v = 0.0;
#pragma unroll
      for (int w = 0; w < kFarrowBlock / 64; ++w) v += sh.s_part[tid][w];
      if (SKY && tid < 2) part_out[tid] = v;
      if (WAVE && tid >= 2) a.gb_part[tid - 2] = v;
    }
  }
}

template <int N, bool SKY>
__global__ __launch_bounds__(kFarrowBlock, 2) void farrow_adjoint_kernel(ProjAdjArgs a) {
  extern __shared__ double lds_dyn[];
  __shared__ FarrowShared sh;
  const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
  farrow_adjoint_tile<N, SKY, false>(a, tile, lds_dyn, sh, a.sky_part + 2 * tile);
}

template <int N, bool SKY, bool WAVE>
__global__ __launch_bounds__(kFarrowBlock, 2) void batch_farrow_adjoint_kernel(BatchAdjArgs a) {
  extern __shared__ double lds_dyn[];
  __shared__ FarrowShared sh;
  const int64_t item = xcd_tile(blockIdx.x, gridDim.x);
  const int64_t b = a.items[2 * item], tile = a.items[2 * item + 1];
  ProjAdjArgs x = batch_proj_args(a, a.tpl[b]);
  x.rows = a.rows;
  if (WAVE) x.gb_part = a.gb_part + 7 * item;
  farrow_adjoint_tile<N, SKY, WAVE>(x, tile, lds_dyn, sh, a.sky_part + 2 * item);
}

template <int N>
hipError_t launch_farrow_adjoint(const ProjAdjArgs& a, hipStream_t s) {
  const int64_t blocks = (a.n_y + kFarrowRuns * a.rows - 1) / (kFarrowRuns * a.rows);
  const bool sky = a.sky_part != nullptr;
  const size_t bytes = farrow_adjoint_doubles(N, sky, false) * sizeof(double);
  if (sky) {
    const hipError_t e = allow_dynamic_lds(farrow_adjoint_kernel<N, true>, bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((farrow_adjoint_kernel<N, true>), dim3((unsigned)blocks), dim3(kFarrowBlock),
                       bytes, s, a);
  } else {
    hipLaunchKernelGGL((farrow_adjoint_kernel<N, false>), dim3((unsigned)blocks), dim3(kFarrowBlock),
                       bytes, s, a);
  }
  return hipGetLastError();
}

template <int N>
hipError_t launch_batch_farrow_adjoint(const BatchAdjArgs& a, int64_t n_items, hipStream_t s) {
  const bool sky = a.sky_part != nullptr;
  const size_t bytes = farrow_adjoint_doubles(N, sky || a.params, a.params) * sizeof(double);
  const dim3 grid((unsigned)n_items), block(kFarrowBlock);
  hipError_t e = allow_dynamic_lds(batch_farrow_adjoint_kernel<N, true, true>, bytes);
  if (e == hipSuccess) e = allow_dynamic_lds(batch_farrow_adjoint_kernel<N, true, false>, bytes);
  if (e != hipSuccess) return e;
  if (a.params)
    hipLaunchKernelGGL((batch_farrow_adjoint_kernel<N, true, true>), grid, block, bytes, s, a);
  else if (sky)
    hipLaunchKernelGGL((batch_farrow_adjoint_kernel<N, true, false>), grid, block, bytes, s, a);
  else
    hipLaunchKernelGGL((batch_farrow_adjoint_kernel<N, false, false>), grid, block, bytes, s, a);
  return hipGetLastError();
}

#define LR_INSTANTIATE_FARROW_ADJ(NT)                                                       \
  template hipError_t launch_farrow_adjoint<NT>(const ProjAdjArgs&, hipStream_t);           \
  template hipError_t launch_batch_farrow_adjoint<NT>(const BatchAdjArgs&, int64_t, hipStream_t);

}  // namespace lr
