// Pixel axes and shapes of the traced grid (Sec. 3.2, eq. "window-kernel"): a, b
// the half differences of the neighbouring projected centres along x and y
// (one-sided at the edges, footnote there), Z = (a a^T + b b^T) / (4 pi).
#pragma once

#include <cmath>

#include "common.hpp"

namespace gpl {

struct PixelAxes {
  float2 a, b;
};

// Axes of point j of an M x M grid (row-major).
__device__ inline PixelAxes pixel_axes(int M, int j, const float* __restrict__ px, const float* __restrict__ py) {
  const int fy = j / M, fx = j - fy * M;
  auto diff = [&](int lo, int hi, float h) -> float2 {  // (p[hi] - p[lo]) * h
    return make_float2((px[hi] - px[lo]) * h, (py[hi] - py[lo]) * h);
  };
  PixelAxes r{make_float2(0.f, 0.f), make_float2(0.f, 0.f)};
  if (M > 1) {
    if (fx == 0) r.a = diff(j, j + 1, 1.f);
    else if (fx == M - 1) r.a = diff(j - 1, j, 1.f);
    else r.a = diff(j - 1, j + 1, 0.5f);
    if (fy == 0) r.b = diff(j, j + M, 1.f);
    else if (fy == M - 1) r.b = diff(j - M, j, 1.f);
    else r.b = diff(j - M, j + M, 0.5f);
  }
  return r;
}

__device__ inline void store_shape(const PixelAxes& p, int N, int j, float* z) {
  const float f = (float)(1.0 / (4.0 * M_PI));
  z[j] = f * (p.a.x * p.a.x + p.b.x * p.b.x);
  z[N + j] = f * (p.a.x * p.a.y + p.b.x * p.b.y);
  z[2 * N + j] = f * (p.a.y * p.a.y + p.b.y * p.b.y);
}

// d a_c / d p_m along one grid line of length M (one-sided differences at the ends).
__device__ inline float axis_coef(int c, int m, int M) {
  if (M == 1) return 0.f;
  if (c == 0) return (m == 1 ? 1.f : 0.f) - (m == 0 ? 1.f : 0.f);
  if (c == M - 1) return (m == M - 1 ? 1.f : 0.f) - (m == M - 2 ? 1.f : 0.f);
  return (m == c + 1 ? 0.5f : 0.f) - (m == c - 1 ? 0.5f : 0.f);
}

// Adjoint of store_shape at point j: gz holds dF/dZ_j as a symmetric matrix gradient;
// Z = (a a^T + b b^T) / (4 pi) gives dF/da = Gbar a / (2 pi), likewise for b.
__device__ inline PixelAxes axes_grad(int M, int j, const float* __restrict__ px, const float* __restrict__ py,
                                      const float* __restrict__ gz) {
  const int N = M * M;
  const PixelAxes ax = pixel_axes(M, j, px, py);
  const float f = (float)(1.0 / (2.0 * M_PI));
  const float gxx = gz[j], gxy = gz[N + j], gyy = gz[2 * N + j];
  return PixelAxes{make_float2(f * fmaf(gxx, ax.a.x, gxy * ax.a.y), f * fmaf(gxy, ax.a.x, gyy * ax.a.y)),
                   make_float2(f * fmaf(gxx, ax.b.x, gxy * ax.b.y), f * fmaf(gxy, ax.b.x, gyy * ax.b.y))};
}

// Adjoint of pixel_axes towards p_m: the axes that depend on it (neighbours c = m-1,
// m, m+1 along the row for a, along the column for b), grad(j) their adjoints.
template <class G>
__device__ inline float2 axes_gather(int M, int m, G grad) {
  const int fy = m / M, fx = m - fy * M;
  float2 s = make_float2(0.f, 0.f);
  for (int c = max(fx - 1, 0); c <= min(fx + 1, M - 1); ++c) {
    const float w = axis_coef(c, fx, M);
    const float2 a = grad(fy * M + c).a;
    s.x = fmaf(w, a.x, s.x);
    s.y = fmaf(w, a.y, s.y);
  }
  for (int c = max(fy - 1, 0); c <= min(fy + 1, M - 1); ++c) {
    const float w = axis_coef(c, fy, M);
    const float2 b = grad(c * M + fx).b;
    s.x = fmaf(w, b.x, s.x);
    s.y = fmaf(w, b.y, s.y);
  }
  return s;
}

}  // namespace gpl
