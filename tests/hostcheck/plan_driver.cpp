// Prints what kernel launches receive, one JSON object per line of standard input.
// "batch": the work plan of a fused batched forward (order, generation, dt, longest
// light times of the projection and of the TDI orbits, group, tile, segment, number
// of templates, their outputs).  "tdi": the taps of the filters of a TDI call and of
// its transpose, 0 for the kernels of single delays (order, generation, dt, longest
// light time, outputs).  The launchers are stubs, and the copies to the device go
// to host memory.
#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#include "../../include/lisaresp.h"
#include "../../paper_2204_06633_amd/csrc/batch_types.hpp"
#include "../../paper_2204_06633_amd/csrc/internal.hpp"

extern "C" {
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
}

namespace lr {
hipError_t run_fused_forward(int, int, int, int, bool, const BatchFwdArgs& a, int, hipStream_t) {
  std::printf("\"F\": %d, \"rows\": %d, \"samples\": %d, \"T_out\": %d, \"halo\": %d, \"HP\": %d, "
              "\"tiles\": %d, \"fir_lo\": %d, \"fir_k\": %d, \"n_fir\": %lld, \"items\": [",
              a.F, a.rows, a.samples, a.T_out, a.halo, a.HP, a.seg_tiles, a.fir_lo, a.fir_k,
              (long long)a.n_fir);
  for (int i = 0; i < a.n_items; ++i)
    std::printf("%s[%d, %d]", i ? ", " : "", a.items[2 * i], a.items[2 * i + 1]);
  std::printf("], ");
  return hipSuccess;
}
hipError_t run_tdi(int, int, const TdiArgs& a, hipStream_t) {
  std::printf("{\"forward\": %d, ", a.fir_k);
  return hipSuccess;
}
hipError_t run_tdi_adjoint(int, int, const TdiAdjArgs& a, hipStream_t) {
  std::printf("\"transpose\": %d}\n", a.fir_k);
  return hipSuccess;
}
}  // namespace lr

static bool tdi() {
  int order, gen;
  double dt, arm, any[1];
  long long n;
  if (std::scanf("%d %d %lf %lf %lld", &order, &gen, &dt, &arm, &n) != 5) return false;
  lr_orbits o{};
  o.dt = 1e7;
  o.n = 100;
  o.coef = any;
  o.L_max = arm;
  o.L_min = 0.98 * arm;
  o.R_max = 1.6e11;
  int64_t f, b;
  if (lr_tdi_padding(&o, order, gen, dt, &f, &b)) return false;
  const auto y = reinterpret_cast<double*>(uintptr_t{1} << 40), g = y + (int64_t{1} << 40);
  return !lr_tdi_combine(&o, 1e6, dt, f + n + b, y, gen, order, LR_AET, f, n, g, nullptr) &&
         !lr_tdi_adjoint(&o, 1e6, dt, f + n + b, gen, order, LR_AET, f, n, g, y, nullptr);
}

int main() {
  int order, gen, group, tile, segment, n;
  double dt, arm_p, arm_t;
  char kind[16];
  while (std::scanf("%15s", kind) == 1) {
    if (std::strcmp(kind, "tdi") == 0) {
      if (!tdi()) return 1;
      continue;
    }
    if (std::scanf("%d %d %lf %lf %lf %d %d %d %d", &order, &gen, &dt, &arm_p, &arm_t, &group,
                   &tile, &segment, &n) != 9)
      return 1;
    double coef[4] = {0.0};
    lr_orbits p{}, t{};
    p.dt = t.dt = 1e7;
    p.n = t.n = 100;
    p.coef = t.coef = coef;
    p.L_max = arm_p;
    t.L_max = arm_t;
    p.L_min = 0.98 * arm_p;
    t.L_min = 0.98 * arm_t;
    p.R_max = t.R_max = 1.6e11;
    p.D_max = 299792458.0 * arm_p;
    p.V_max = 3e4;
    int64_t fp, bp, ft, bt;
    if (lr_projection_padding(&p, order, dt, &fp, &bp) ||
        lr_tdi_padding(&t, order, gen, dt, &ft, &bt))
      return 1;
    std::vector<lr_template> v(n);
    int64_t h = 0, o = 0;
    for (auto& T : v) {
      long long n_out;
      if (std::scanf("%lld", &n_out) != 1) return 1;
      T.n_out = n_out;
      T.out_start = fp + ft;
      T.n_h = fp + ft + n_out + bt + bp;
      T.h_offset = h;
      T.out_offset = o;
      h += T.n_h;
      o += 3 * n_out;
    }
    const size_t ws = lr_batch_workspace(v.data(), n, &t, dt, order, gen, LR_AET, group, tile,
                                         segment, 1);
    std::vector<double> store(ws / sizeof(double) + 1);
    lr_batch b{};
    double any[2];
    std::printf("{\"workspace\": %zu, ", ws);
    const int st = lr_batch_prepare(v.data(), n, &p, &t, 1e8, dt, order, gen, LR_AET, group, tile,
                                    segment, 1, store.data(), ws, &b, nullptr);
    if (st == LR_OK) lr_response(&b, any, any, any, any, nullptr);
    std::printf("\"status\": %d}\n", st);
  }
  return 0;
}
