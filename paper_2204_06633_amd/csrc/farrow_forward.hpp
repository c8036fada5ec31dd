// Link responses from polynomials per stencil base (farrow.hpp; FP64, gfx950).
//
// A workgroup of BLOCK lanes takes a run of up to BLOCK minus the spread of
// the nine positions consecutive link samples, so that BLOCK stencil bases
// cover it:
//   A. lane = link sample: geometry, fraction and integer part per position;
//   B. lane = stencil base: coefficients of h+ and hx from the window in LDS,
//      then position by position the value at the link sample it serves, into
//      that sample's LDS slots (which held its fraction);
//   C. lane = link sample: the links from the nine values.
// G positions at a time go through LDS.  A value depends on its stencil and
// fraction alone, not on how link samples are dealt to runs.
//
// Bound by FP64 issue (VALU 75 % busy at three waves per SIMD; 64 registers of
// coefficients rule out four).  Order 25, dt = 10 s, against nine weight
// sequences per link sample shared by two samples of a lane: 3,155,760 samples
// 250 -> 170 us, 8640 samples 17 -> 13 us; in the fused batched forward, 32
// templates of 1.5 million outputs, 6.40 -> 5.27 ms.
#pragma once

#include "farrow.hpp"

namespace lr {

// PAD: positions up to this far apart take the quick path of phase B, in which
// a base's link sample is its lane minus up to PAD: what lies before a row's
// first sample in LDS is never read.
template <int N, int BLOCK, int G, int PAD>
struct FarrowForward {
  static constexpr int LD = BLOCK + PAD;
  double val[2][G * LD];                       // fraction, then h+; hx
  double2 win[BLOCK + N];
  int lo[BLOCK / 64][9], hi[BLOCK / 64][9];    // per wave: integer parts of the positions

  // The six links of link sample ti0 + t, t = the lane, at orbit time
  // t_off + (ti0 + t) dt and h-index hq0 + t; lanes from n on repeat the last
  // one.  Contains barriers.
  __device__ __forceinline__ void project(const OrbitView& orb, double t_off, int64_t ti0,
                                          double dt, double inv_dt, const HSource& hs,
                                          int64_t hq0, const Sky& sk, int t, int n,
                                          double (&y)[6]);
};

template <int N, int BLOCK, int G, int PAD>
__device__ __forceinline__ void FarrowForward<N, BLOCK, G, PAD>::project(
    const OrbitView& orb, double t_off, int64_t ti0, double dt, double inv_dt, const HSource& hs,
    int64_t hq0, const Sky& sk, int t, int n, double (&y)[6]) {
  constexpr int H = N / 2, D = FarrowTable<N>::D, W = BLOCK / 64;
  const int lane = t & 63, wv = t >> 6;
  const int rel = min(t, n - 1);

  // A.
  double xip[3], xic[3], kn[3], u[9];
  int f[9], wlo = 0;                           // lane p < 9: the wave's range of position p
  {
    LinkGeom g;
    link_geometry(orb, t_off + (double)(ti0 + rel) * dt, sk, g);
    int differ = 0;
#pragma unroll
    for (int p = 0; p < 9; ++p) {
      f[p] = split_centred(position_delay(g, p), inv_dt, u[p]);
      const int a = __builtin_amdgcn_readfirstlane(f[p]);
      differ |= f[p] ^ a;
      wlo = lane == p ? a : wlo;
    }
    int whi = wlo;
    if (__any(differ)) {
#pragma unroll
      for (int p = 0; p < 9; ++p) {
        const int a = wave_min(f[p]), b = wave_max(f[p]);
        wlo = lane == p ? a : wlo;
        whi = lane == p ? b : whi;
      }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      xip[k] = g.xip[k];
      xic[k] = g.xic[k];
      kn[k] = g.kn[k];
    }
    if (lane < 9) {
      lo[wv][lane] = wlo;
      hi[wv][lane] = whi;
    }
  }
  __syncthreads();                             // also: the previous run is done with LDS
  const int pl = min(lane, 8);
  int whi = hi[0][pl];
  wlo = lo[0][pl];
#pragma unroll
  for (int w = 1; w < W; ++w) {
    wlo = min(wlo, lo[w][pl]);
    whi = max(whi, hi[w][pl]);
  }
  const bool uniform = __all(wlo == whi);      // one integer part per position
  int plo[9], jlo = 1 << 30, jhi = -(1 << 30), drift = 0;
#pragma unroll
  for (int p = 0; p < 9; ++p) {
    plo[p] = __builtin_amdgcn_readlane(wlo, p);
    const int phi = __builtin_amdgcn_readlane(whi, p);
    jlo = min(jlo, plo[p]);
    jhi = max(jhi, phi);
    drift = max(drift, phi - plo[p]);
  }

  double hp[9], hc[9];
  if (n + jhi - jlo <= BLOCK && drift < 256) {
    const int nj = n + jhi - jlo;
    const int64_t j0 = hq0 + jlo - (H - 1);    // h-index of window element 0
    for (int k = t; k < nj + N - 1; k += BLOCK) {
      int64_t j = j0 + k;
      j = j < 0 ? 0 : (j > hs.n_h - 1 ? hs.n_h - 1 : j);
      win[k] = hs.at(j);
    }
    const bool fast = uniform && jhi - jlo <= PAD;
    auto put = [&](int first) {
#pragma unroll
      for (int p = first; p < 9 && p < first + G; ++p) val[0][(p - first) * LD + PAD + t] = u[p];
    };
    unsigned fb[3] = {0, 0, 0};                // integer parts minus the position's smallest
#pragma unroll
    for (int p = 0; p < 9; ++p) fb[p / 4] |= (unsigned)(f[p] - plo[p]) << (8 * (p % 4));
    put(0);
    __syncthreads();                           // window, fractions

    // B.
    double cp[D + 1], cc[D + 1];
    farrow_coefs<N>(win + min(t, nj - 1), cp, cc);
    // the integer parts go where the window was
    unsigned char* fs = reinterpret_cast<unsigned char*>(win);
    static_assert(sizeof(win) >= 9 * BLOCK, "integer parts fit the window");
    auto horner = [&](double x, double& vp, double& vc) {
      vp = cp[D];
      vc = cc[D];
#pragma unroll
      for (int m = D - 1; m >= 0; --m) {
        vp = fma(vp, x, cp[m]);
        vc = fma(vc, x, cc[m]);
      }
    };
#pragma unroll
    for (int first = 0; first < 9; first += G) {
      constexpr int last = 9;
      const int end = first + G < last ? first + G : last;
      if (first > 0) {
        put(first);
        __syncthreads();
      }
      if (fast) {
        // base t serves link sample t + jlo - f: past the ends of the run it
        // works on what no one reads
        double x[G];
#pragma unroll
        for (int p = first; p < end; ++p)
          x[p - first] = val[0][(p - first) * LD + PAD + t + (jlo - plo[p])];
#pragma unroll
        for (int p = first; p < end; ++p) {
          double* v = &val[0][(p - first) * LD + PAD + t + (jlo - plo[p])];
          double vp, vc;
          horner(x[p - first], vp, vc);
          v[0] = vp;
          v[G * LD] = vc;
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
        if (first == 0) {
          __syncthreads();
#pragma unroll
          for (int p = 0; p < 9; ++p)
            fs[p * BLOCK + t] = (unsigned char)(fb[p / 4] >> (8 * (p % 4)));
          __syncthreads();
        }
#pragma unroll 1
        for (int p = first; p < end; ++p) {
          const int a = __builtin_amdgcn_readlane(wlo, p), b = __builtin_amdgcn_readlane(whi, p);
#pragma unroll 1
          for (int k = a; k <= b; ++k) {
            const int r = t + jlo - k, rc = min(max(r, 0), n - 1);
            const bool ok = r == rc && (int)fs[p * BLOCK + rc] == k - a;
            double* v = &val[0][(p - first) * LD + PAD + rc];
            double vp, vc;
            horner(ok ? v[0] : 0.0, vp, vc);
            if (ok) {
              v[0] = vp;
              v[G * LD] = vc;
            }
          }
        }
      }
      __syncthreads();

      // C.
#pragma unroll
      for (int p = first; p < end; ++p) {
        hp[p] = val[0][(p - first) * LD + PAD + rel];
        hc[p] = val[1][(p - first) * LD + PAD + rel];
      }
      if (end < 9) __syncthreads();
    }
  } else {
    // Positions further apart than the workgroup's bases reach (very small dt
    // or extreme orbits): each stencil from the source, indices clamped.
#pragma unroll 1
    for (int q = 0; q < 9; ++q) {
      double eps = u[0];
      int sh = f[0];
#pragma unroll
      for (int p = 1; p < 9; ++p) {
        eps = p == q ? u[p] : eps;
        sh = p == q ? f[p] : sh;
      }
      LagrangeStream<N> st(eps + 0.5);
      double vp = 0.0, vc = 0.0;
#pragma unroll 2
      for (int m = 0; m < N; ++m) {
        int64_t j = hq0 + rel + sh - (H - 1) + m;
        j = j < 0 ? 0 : (j > hs.n_h - 1 ? hs.n_h - 1 : j);
        const double2 v = hs.at(j);
        st.tap(m);
        vp = st.step(vp, v.x, m);
        vc = st.step(vc, v.y, m);
      }
      vp = st.finish(vp);
      vc = st.finish(vc);
#pragma unroll
      for (int p = 0; p < 9; ++p) {
        hp[p] = p == q ? vp : hp[p];
        hc[p] = p == q ? vc : hc[p];
      }
    }
    __syncthreads();                           // lo, hi read before the next run's
  }
#pragma unroll
  for (int l = 0; l < 6; ++l) {
    const int arm = kArm[l], r = kLinkRecv[l] - 1;
    y[l] = 0.5 * fma(xip[arm], hp[3 + l] - hp[r], xic[arm] * (hc[3 + l] - hc[r])) *
           fast_rcp(1.0 - kDir[l] * kn[arm]);
  }
}

// Waves per SIMD that the projection's registers leave room for: three, or more where
// a build asks for more (four spill the coefficients: 3,155,760 samples of order 25
// 347 us against 252).
#ifndef LR_PROJ_MIN_WAVES
#define LR_PROJ_MIN_WAVES 1
#endif
constexpr int kProjWaves = LR_PROJ_MIN_WAVES > 3 ? LR_PROJ_MIN_WAVES : 3;

template <int N>
__global__ __launch_bounds__(kFarrowBlock, kProjWaves) void farrow_project_kernel(ProjArgs a) {
  __shared__ FarrowForward<N, kFarrowBlock, 9, kFarrowSpread> sh;
  __shared__ double s_trig[2][2];
  const SkyTrig tr = load_sky(a.sky, s_trig);
  const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
  const int64_t end = min(a.n_y, (tile + 1) * a.runs * a.rows);
#pragma unroll 1
  for (int64_t r0 = tile * a.runs * a.rows; r0 < end; r0 += a.rows) {
    int t = threadIdx.x;                       // opaque: nothing hoisted out of the loop
    asm volatile("" : "+v"(t));
    const int n = (int)min((int64_t)a.rows, end - r0);
    double y[6];
    sh.project(a.orb, a.t_off, a.y_start + r0, a.dt, a.inv_dt,
               HSource::arrays(a.hp, a.hc, a.n_h), a.y_start + r0,
               sky_from_trig(tr.sl, tr.cl, tr.sb, tr.cb), t, n, y);
    if (t < n)
#pragma unroll
      for (int l = 0; l < 6; ++l) a.y[(int64_t)l * a.n_y + r0 + t] = y[l];
  }
}

template <int N>
hipError_t launch_project(const ProjArgs& a, hipStream_t s) {
  const int64_t run = (int64_t)a.runs * a.rows, blocks = (a.n_y + run - 1) / run;
  hipLaunchKernelGGL(farrow_project_kernel<N>, dim3((unsigned)blocks), dim3(kFarrowBlock), 0, s, a);
  return hipGetLastError();
}

#define LR_INSTANTIATE_FARROW_FWD(NT) \
  template hipError_t launch_project<NT>(const ProjArgs&, hipStream_t);

}  // namespace lr
