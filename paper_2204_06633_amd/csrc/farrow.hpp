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

// The numbers of mirrored pair i: j < 8 the coefficient of u^(2 j) per sum,
// 8 + j that of u^(2 j + 1) per difference.
template <int N>
struct FarrowRows {
  double w[N / 2][16];
};

template <int N>
constexpr FarrowRows<N> farrow_rows_of() {
  FarrowRows<N> m{};
  for (int j = 0; j <= FarrowTable<N>::D; ++j)
    for (int i = 0; i < N / 2; ++i)
      m.w[i][(j & 1) * 8 + j / 2] =
          j % 2 == 0 ? FarrowTable<N>::e[j / 2][i] : FarrowTable<N>::o[j / 2][i];
  return m;
}

template <int N>
__constant__ FarrowRows<N> kFarrowRows = farrow_rows_of<N>();

// Pair i's numbers into scalar registers.  The opaque index keeps the loads
// where they stand: the compiler would otherwise hoist all 16 N / 2 of them
// out of the callers' loops.  Of the ways to feed them to the FMAs, literals
// cost two scalar moves each and broadcasts from a lane (DPP) issue at 24-28
// of the 32-34 10^12 FMA/s that scalar operands reach (projection of 3,155,760
// samples at order 25: 183 against 173 us).
template <int N>
__device__ __forceinline__ void farrow_row(int i, double (&w)[16]) {
  int o = 16 * i;
  asm volatile("" : "+s"(o));
  const auto r =
      (const __attribute__((address_space(4))) double*)&kFarrowRows<N>.w[0][0] + o;
#pragma unroll
  for (int j = 0; j < 16; ++j) w[j] = r[j];
}

// Coefficients of u^0 .. u^D of both polarisations from the stencil
// win[0 .. N - 1].
template <int N>
__device__ __forceinline__ void farrow_coefs(const double2* win, double (&p)[kFarrowCoefs<N>],
                                             double (&c)[kFarrowCoefs<N>]) {
  using T = FarrowTable<N>;
  constexpr int H = N / 2, D = T::D;
  if constexpr (D == 15) {
    double2 a = win[H], b = win[H - 1];
    double w[16];
    farrow_row<N>(0, w);
#pragma unroll
    for (int i = 0; i < H; ++i) {
      // the next pair is read while this one is summed, and no earlier: all
      // reads at the top would spill
      const int n = i + 1 < H ? i + 1 : i;
      const double2 an = win[H + n], bn = win[H - 1 - n];
      double v[16];
      farrow_row<N>(n, v);
      __builtin_amdgcn_sched_barrier(0);
      const double ex = a.x + b.x, ey = a.y + b.y, ox = a.x - b.x, oy = a.y - b.y;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        p[2 * j] = i == 0 ? w[j] * ex : fma(w[j], ex, p[2 * j]);
        c[2 * j] = i == 0 ? w[j] * ey : fma(w[j], ey, c[2 * j]);
        p[2 * j + 1] = i == 0 ? w[8 + j] * ox : fma(w[8 + j], ox, p[2 * j + 1]);
        c[2 * j + 1] = i == 0 ? w[8 + j] * oy : fma(w[8 + j], oy, c[2 * j + 1]);
      }
      __builtin_amdgcn_sched_barrier(0);
      a = an;
      b = bn;
#pragma unroll
      for (int j = 0; j < 16; ++j) w[j] = v[j];
    }
    // computed here: sunk into a caller's branches, the sums would leave all
    // rows loaded before them and spilled (adjoint with sky gradient of 3,155,760
    // samples: 483 against 441 us)
#pragma unroll
    for (int j = 0; j <= D; ++j) asm volatile("" : "+v"(p[j]), "+v"(c[j]));
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
  double w[16];
  if constexpr (D == 15) farrow_row<N>(0, w);
#pragma unroll
  for (int i = 0; i < H; ++i) {
    double ep = 0.0, ec = 0.0, op = 0.0, oc = 0.0;
    if constexpr (D == 15) {
      double v[16];
      farrow_row<N>(i + 1 < H ? i + 1 : i, v);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        ep = fma(w[j], p[2 * j], ep);
        ec = fma(w[j], c[2 * j], ec);
        op = fma(w[8 + j], p[2 * j + 1], op);
        oc = fma(w[8 + j], c[2 * j + 1], oc);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 16; ++j) w[j] = v[j];
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
