// Lagrange interpolation at many positions as polynomials per sample (FP64,
// gfx950).
//
// Between two samples the interpolant (Sec. IV.E) is one polynomial of degree
// N - 1 in the fraction eps, whatever the position: its coefficients are fixed
// linear combinations of the stencil's N samples.  A lane that owns the
// stencil base J forms them once (taps in mirrored pairs: the even
// coefficients of u = eps - 1/2 act on the sums, the odd ones on the
// differences) and then serves every link sample and position whose retarded
// time falls into [J, J + 1): nine of them on average, h+ and hx each, by
// Horner's rule.  Above degree 15 the coefficients are below rounding on
// |u| <= 1/2 and are dropped (build.py: at most 2.5e-17 of the largest
// sample).  Per link sample at order 25: 2 x (208 + 26) operations for the
// coefficients and 9 x 2 x 15 for the positions, against 9 x 26 x 6.5 for
// nine weight sequences; with derivatives 9 x 2 x 29 against 9 x 26 x 19.
#pragma once

#include "forward_kernels.hpp"
#include "farrow_tables.hpp"

namespace lr {

template <int N>
constexpr int kFarrowCoefs = FarrowTable<N>::D + 1;

// The numbers of mirrored pair i in the 16 lanes of a DPP row: lane j < 8 the
// coefficient of u^(2 j) per sum, lane 8 + j that of u^(2 j + 1) per
// difference.  An FMA takes its number by row_newbcast: as a literal each would
// cost two scalar moves, which take issue slots from the FMAs at two waves per
// SIMD.
template <int N>
struct FarrowLanes {
  double w[N / 2][16];
};

template <int N>
constexpr FarrowLanes<N> farrow_lanes() {
  FarrowLanes<N> m{};
  for (int j = 0; j <= FarrowTable<N>::D; ++j)
    for (int i = 0; i < N / 2; ++i)
      m.w[i][(j & 1) * 8 + j / 2] =
          j % 2 == 0 ? FarrowTable<N>::e[j / 2][i] : FarrowTable<N>::o[j / 2][i];
  return m;
}

template <int N>
__constant__ FarrowLanes<N> kFarrowLanes = farrow_lanes<N>();

// p[j], c[j] += number first + j/2 of w's row times x, y, for even j (or odd j).
__device__ __forceinline__ void farrow_even(double (&p)[16], double (&c)[16], double w, double x,
                                            double y) {
  asm(
      "s_nop 1\n"
      "v_fmac_f64_dpp %0, %16, %17 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %8, %16, %18 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %16, %17 row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %9, %16, %18 row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %16, %17 row_newbcast:2 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %10, %16, %18 row_newbcast:2 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %16, %17 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %11, %16, %18 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %4, %16, %17 row_newbcast:4 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %12, %16, %18 row_newbcast:4 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %5, %16, %17 row_newbcast:5 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %13, %16, %18 row_newbcast:5 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %6, %16, %17 row_newbcast:6 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %14, %16, %18 row_newbcast:6 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %7, %16, %17 row_newbcast:7 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %15, %16, %18 row_newbcast:7 row_mask:0xf bank_mask:0xf\n"
      : "+v"(p[0]), "+v"(p[2]), "+v"(p[4]), "+v"(p[6]), "+v"(p[8]), "+v"(p[10]), "+v"(p[12]), "+v"(p[14]),
        "+v"(c[0]), "+v"(c[2]), "+v"(c[4]), "+v"(c[6]), "+v"(c[8]), "+v"(c[10]), "+v"(c[12]), "+v"(c[14])
      : "v"(w), "v"(x), "v"(y));
}
__device__ __forceinline__ void farrow_odd(double (&p)[16], double (&c)[16], double w, double x,
                                           double y) {
  asm(
      "s_nop 1\n"
      "v_fmac_f64_dpp %0, %16, %17 row_newbcast:8 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %8, %16, %18 row_newbcast:8 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %16, %17 row_newbcast:9 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %9, %16, %18 row_newbcast:9 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %16, %17 row_newbcast:10 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %10, %16, %18 row_newbcast:10 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %16, %17 row_newbcast:11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %11, %16, %18 row_newbcast:11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %4, %16, %17 row_newbcast:12 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %12, %16, %18 row_newbcast:12 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %5, %16, %17 row_newbcast:13 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %13, %16, %18 row_newbcast:13 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %6, %16, %17 row_newbcast:14 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %14, %16, %18 row_newbcast:14 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %7, %16, %17 row_newbcast:15 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %15, %16, %18 row_newbcast:15 row_mask:0xf bank_mask:0xf\n"
      : "+v"(p[1]), "+v"(p[3]), "+v"(p[5]), "+v"(p[7]), "+v"(p[9]), "+v"(p[11]), "+v"(p[13]), "+v"(p[15]),
        "+v"(c[1]), "+v"(c[3]), "+v"(c[5]), "+v"(c[7]), "+v"(c[9]), "+v"(c[11]), "+v"(c[13]), "+v"(c[15])
      : "v"(w), "v"(x), "v"(y));
}
// x, y += sum over even (odd) j of number j of w's row times p[j], c[j].
__device__ __forceinline__ void farrow_even_t(const double (&p)[16], const double (&c)[16],
                                              double w, double& x, double& y) {
  asm(
      "s_nop 1\n"
      "v_fmac_f64_dpp %0, %2, %3 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %2, %11 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %2, %4 row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %2, %12 row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %2, %5 row_newbcast:2 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %2, %13 row_newbcast:2 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %2, %6 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %2, %14 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %2, %7 row_newbcast:4 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %2, %15 row_newbcast:4 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %2, %8 row_newbcast:5 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %2, %16 row_newbcast:5 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %2, %9 row_newbcast:6 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %2, %17 row_newbcast:6 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %2, %10 row_newbcast:7 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %2, %18 row_newbcast:7 row_mask:0xf bank_mask:0xf\n"
      : "+v"(x), "+v"(y)
      : "v"(w), "v"(p[0]), "v"(p[2]), "v"(p[4]), "v"(p[6]), "v"(p[8]), "v"(p[10]), "v"(p[12]), "v"(p[14]),
        "v"(c[0]), "v"(c[2]), "v"(c[4]), "v"(c[6]), "v"(c[8]), "v"(c[10]), "v"(c[12]), "v"(c[14]));
}
__device__ __forceinline__ void farrow_odd_t(const double (&p)[16], const double (&c)[16],
                                             double w, double& x, double& y) {
  asm(
      "s_nop 1\n"
      "v_fmac_f64_dpp %0, %2, %3 row_newbcast:8 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %2, %11 row_newbcast:8 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %2, %4 row_newbcast:9 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %2, %12 row_newbcast:9 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %2, %5 row_newbcast:10 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %2, %13 row_newbcast:10 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %2, %6 row_newbcast:11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %2, %14 row_newbcast:11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %2, %7 row_newbcast:12 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %2, %15 row_newbcast:12 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %2, %8 row_newbcast:13 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %2, %16 row_newbcast:13 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %2, %9 row_newbcast:14 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %2, %17 row_newbcast:14 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %2, %10 row_newbcast:15 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %2, %18 row_newbcast:15 row_mask:0xf bank_mask:0xf\n"
      : "+v"(x), "+v"(y)
      : "v"(w), "v"(p[1]), "v"(p[3]), "v"(p[5]), "v"(p[7]), "v"(p[9]), "v"(p[11]), "v"(p[13]), "v"(p[15]),
        "v"(c[1]), "v"(c[3]), "v"(c[5]), "v"(c[7]), "v"(c[9]), "v"(c[11]), "v"(c[13]), "v"(c[15]));
}

// Coefficients of u^0 .. u^D of both polarisations from the stencil
// win[0 .. N - 1].
template <int N>
__device__ __forceinline__ void farrow_coefs(const double2* win, double (&p)[kFarrowCoefs<N>],
                                             double (&c)[kFarrowCoefs<N>]) {
  using T = FarrowTable<N>;
  constexpr int H = N / 2, D = T::D;
  if constexpr (D == 15) {
    const double* w = &kFarrowLanes<N>.w[0][threadIdx.x & 15];
#pragma unroll
    for (int j = 0; j <= D; ++j) p[j] = c[j] = 0.0;
    double2 a = win[H], b = win[H - 1];
    double x = w[0];
#pragma unroll
    for (int i = 0; i < H; ++i) {
      // the next pair is read while this one is summed, and no earlier: all
      // reads at the top would spill
      const int n = i + 1 < H ? i + 1 : i;
      const double2 an = win[H + n], bn = win[H - 1 - n];
      const double xn = w[16 * n];
      __builtin_amdgcn_sched_barrier(0);
      farrow_even(p, c, x, a.x + b.x, a.y + b.y);
      farrow_odd(p, c, x, a.x - b.x, a.y - b.y);
      __builtin_amdgcn_sched_barrier(0);
      a = an;
      b = bn;
      x = xn;
    }
  } else {
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const double2 a = win[H + i], b = win[H - 1 - i];
#pragma unroll
      for (int j = 0; j <= D; ++j) {
        const double w = j % 2 == 0 ? T::e[j / 2][i] : T::o[j / 2][i];
        const double x = j % 2 == 0 ? a.x + b.x : a.x - b.x;
        const double y = j % 2 == 0 ? a.y + b.y : a.y - b.y;
        p[j] = i == 0 ? w * x : fma(w, x, p[j]);
        c[j] = i == 0 ? w * y : fma(w, y, c[j]);
      }
    }
  }
}

// The transpose: put(k, gp, gc), k = 0 .. N - 1, with the gradients of the
// stencil's samples from those of the coefficients.
template <int N, class Put>
__device__ __forceinline__ void farrow_transpose(const double (&p)[kFarrowCoefs<N>],
                                                 const double (&c)[kFarrowCoefs<N>],
                                                 const Put& put) {
  using T = FarrowTable<N>;
  constexpr int H = N / 2, D = T::D;
  const double* row = &kFarrowLanes<N>.w[0][threadIdx.x & 15];
  double x = row[0];
#pragma unroll
  for (int i = 0; i < H; ++i) {
    double ep = 0.0, ec = 0.0, op = 0.0, oc = 0.0;
    if constexpr (D == 15) {
      const double xn = row[16 * (i + 1 < H ? i + 1 : i)];
      __builtin_amdgcn_sched_barrier(0);
      farrow_even_t(p, c, x, ep, ec);
      farrow_odd_t(p, c, x, op, oc);
      x = xn;
    } else {
#pragma unroll
      for (int j = 0; j <= D; ++j) {
        const double w = j % 2 == 0 ? T::e[j / 2][i] : T::o[j / 2][i];
        double& x = j % 2 == 0 ? ep : op;
        double& y = j % 2 == 0 ? ec : oc;
        x = fma(w, p[j], x);
        y = fma(w, c[j], y);
      }
    }
    put(H + i, ep + op, ec + oc);
    put(H - 1 - i, ep - op, ec - oc);
  }
}

}  // namespace lr
