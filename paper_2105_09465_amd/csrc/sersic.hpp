// Circular Sersic mean function at one point (sersic.hip, vigp.hip).
#pragma once

#include "common.hpp"

namespace gpl {

struct SersicF {
  float I_e, inv_Re, inv_n, bn_log2e, bn, xs, ys;
};
SersicF make_sersic(const gpl_source* s);
int check_source(const gpl_source* s);

// (r/R_e)^(1/n) via exp2(log2(.)/n); r = 0 gives exp2(-inf) = 0.
__device__ inline float sersic_shape(const SersicF& S, float dx, float dy, float& t) {
  const float r = sqrtf(dx * dx + dy * dy);
  t = exp2f(log2f(r * S.inv_Re) * S.inv_n);
  return S.I_e * exp2f(S.bn_log2e * (1.f - t));
}

// d mu / d p = factor (dx, dy): -mu b_n/n (r/R_e)^(1/n) / r^2, zero at r = 0 by convention.
__device__ inline float sersic_slope(const SersicF& S, float dx, float dy) {
  float t;
  const float m = sersic_shape(S, dx, dy, t);
  const float r2 = dx * dx + dy * dy;
  return r2 > 0.f ? -m * S.bn * S.inv_n * t / r2 : 0.f;
}

}  // namespace gpl
