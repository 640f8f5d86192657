// Mixed-precision iterative refinement: outer scaling and update kernels.
#pragma once

#include "common.hpp"

namespace its {

// ------------------------------------------------- mixed-precision refinement
// Outer step: rh = (float)(r/rn), d = 0, rh.rh; then (after the inner CG)
// x += rn * d in double.

// p starts as 0: the second member of the {rh, p} pairs, or a vector of its own.
template <bool Pairs>
__global__ void __launch_bounds__(kBlock) k_ir_scale(int32_t n, const double *__restrict__ r,
                                                     float *__restrict__ rh, float *__restrict__ p,
                                                     float *__restrict__ d, Reduce *R, double rn) {
  Dot2 a;
  for_rows(n, [&](int32_t i) {
    const float v = float(r[i] / rn);
    if constexpr (Pairs) {
      float2_t o;
      o.x = v;
      o.y = 0.0f;
      reinterpret_cast<float2_t *>(rh)[i] = o;
    } else {
      rh[i] = v;
      p[i] = 0.0f;
    }
    d[i] = 0.0f;
    a.add(double(v), double(v));
  });
  DD v[1] = {a.get()};
  block_partial<1>(v, R);
}

__global__ void __launch_bounds__(kBlock) k_ir_update(int32_t n, double *__restrict__ x,
                                                      const float *__restrict__ d, double rn) {
  for_rows(n, [&](int32_t i) { st_nt(x + i, fma(rn, double(ld_nt(d + i)), ld_nt(x + i))); });
}

}  // namespace its
