// Adjoint of the kernel-matrix product with kernel tiles recomputed (the paper
// differentiates its matrix-free product automatically, Sec. 3.3; here the
// adjoint is written out). For F = sum_c w_c a_c^T K b_c with
// K_ij = a^2 exp(-|p_i - p_j|^2 / (2 l^2)) (eq. "grbf"):
//   s_ij     = sum_c w_c (a_ic b_jc + a_jc b_ic)
//   dF/dp_i  = -(1/l^2) sum_j K_ij s_ij (p_i - p_j)
//   dF/dl    = (1/2) sum_ij K_ij s_ij |p_i - p_j|^2 / l^3
//   dF/da    = sum_ij K_ij s_ij / a          (= 2F/a)
// The points are taken in the order of the product's tile plan and the pairs are
// the plan's: (16-point subtile, 32-point chunk) pairs of boxes with s2 g^2 <
// kSkipBackward for their gap g, split over the waves by cost. Beyond that every
// kernel value is at most a^2 2^-36, so each skipped term K s (p_i - p_j) is below
// 2^-36 of the same term at kernel value a^2 (the product's forms treat these
// values in the same way).
//
// s_ij is a contraction over the columns, P_i . Q_j with P = (w a, w b), Q = (b, a):
// FP32 MFMA (v_mfma_f32_16x16x4_f32) with the sources j as rows and the points i as
// columns of its result, so that a lane holds four j of one i and the sums over j
// stay in registers. They are FP64 moments of K s about the row tile's first
// point, sum K s (1, x_j, y_j, x_j^2 + y_j^2), from which dF/dp_i, dF/dl and dF/da of
// a row follow at the end: one conversion and four FP64 operations a pair (the
// differences in FP64 take three more conversions).
//
// The moments cancel: their sum of K s d^2 has an error of some 2^-53 E^2 sum |K s| for
// a tile of extent E, against terms of l^2 sum |K s|. Up to E^2 s2 = kWideTile = 2^20
// (E some 1,200 l) that is 2^-33 of the sum, below the terms' own FP32 rounding; a
// wider tile (a point of its own far away, two clusters that share a tile, a
// non-finite coordinate, whose box is infinite) adds up the differences. A point's own
// term and those of its duplicates, which have no difference, leave some 2^-53 E |K s| in
// the moments: a gradient below that (of a point whose neighbours' K are below 1e-10) is
// rounding.
//
// Bound by VALU issue (six FP32, one exp, one conversion and four FP64
// instructions a pair) beside 9 MFMAs for 256 pairs at 17 columns: 93 us at 40,000
// traced points and 17 columns (91 without the look at the tile's box). The previous
// kernel (s_ij by FMAs from LDS-staged columns, 512-row blocks against 32-point chunks)
// took 650-730 us for 16 columns of 40,000 points and another 260 us for the seventeenth.
#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "internal.hpp"
#include "tileplan.hpp"

namespace gpl {

constexpr int kMaxPass = 18;  // column pairs per pass
constexpr float kSkipBackward = kSkipFp32;
constexpr int kBwdSums = 4;   // sums of a row: gx, gy (without -1/l^2), K s d^2, K s
constexpr double kWideTile = 1 << 20;  // extent^2 s2 of a row tile from which differences are summed

// MFMA steps of a pass of nc column pairs: step s of lane group g takes entry
// g S + s of the 2 nc entries of P and Q (zero padded to 4 S).
static int bwd_steps(int nc) {
  const int s = cdiv(nc, 2);
  return s > 8 ? 9 : s > 4 ? 8 : s > 2 ? 4 : s;
}
// Floats of one lane's entries in memory: a power of two or a multiple of four.
__host__ __device__ constexpr int bwd_stride(int S) { return S > 8 ? 12 : S; }
// Entries of sorted point j in lane group g.
__host__ __device__ inline size_t bwd_at(int j, int g, int stride) {
  return ((size_t)((j >> 4) * 4 + g) * 16 + (j & 15)) * stride;
}

struct WChunk {
  float w[kMaxPass];  // weights of the column pairs of one pass
};

typedef float bwd_f4 __attribute__((ext_vector_type(4)));

// The S entries of one lane.
template <int S>
__device__ __forceinline__ void bwd_load(float (&v)[S], const float* __restrict__ p) {
  if (S == 1) {
    v[0] = p[0];
  } else if (S == 2) {
    const float2 t = *reinterpret_cast<const float2*>(p);
    v[0] = t.x;
    v[1 % S] = t.y;
  } else {
#pragma unroll
    for (int q = 0; q < S / 4; ++q) {
      const bwd_f4 t = *reinterpret_cast<const bwd_f4*>(p + 4 * q);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[(4 * q + k) % S] = t[k];
    }
    if (S % 4 == 1) v[S - 1] = p[S - 1];
  }
}

// P and Q of the columns c0 .. c0 + nc in the plan's order, zeros past n: thread
// (sorted point, lane group), its S entries of both, so that the lanes of a wave
// write one run of memory.
template <int S>
__global__ __launch_bounds__(256) void bwd_gather_kernel(int n, int npad, int nc, int c0, const int* __restrict__ perm,
                                                         const float* __restrict__ A, int lda,
                                                         const float* __restrict__ Bv, int ldb, WChunk w,
                                                         float* __restrict__ P, float* __restrict__ Q) {
  constexpr int stride = bwd_stride(S);
  const int o = blockIdx.x * 256 + threadIdx.x;  // (16-point group, lane group, point of the group)
  if (o >= 4 * npad) return;
  const int g = (o >> 4) & 3, j = (o >> 6) * 16 + (o & 15);
  const bool live = j < n;
  const int i = live ? perm[j] : 0;
  float p[S], q[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int k = g * S + s, c = k < 2 * S ? k : k - 2 * S;  // entries (w a, b), then (w b, a)
    const bool ok = live && c < nc;
    const float a = ok ? A[(size_t)(c0 + c) * lda + i] : 0.f, b = ok ? Bv[(size_t)(c0 + c) * ldb + i] : 0.f;
    p[s] = w.w[min(c, kMaxPass - 1)] * (k < 2 * S ? a : b);
    q[s] = k < 2 * S ? b : a;
  }
  float *dp = P + (size_t)o * stride, *dq = Q + (size_t)o * stride;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    dp[s] = p[s];
    dq[s] = q[s];
  }
}

// A row tile's sums over the list positions [kb, ke): of K s, and its moments about
// (cx, cy) or (kWide) its products with the differences.
template <int S, bool kWide>
__device__ __forceinline__ void bwd_accumulate(const TilePlan& T, float s2, const float* __restrict__ Q,
                                               const uint32_t* __restrict__ lst, int kb, int ke,
                                               const float (&xi)[kSubsPerTile], const float (&yi)[kSubsPerTile],
                                               const float (&pf)[kSubsPerTile][S], double cx, double cy,
                                               double (&s0)[kSubsPerTile], double (&sx)[kSubsPerTile],
                                               double (&sy)[kSubsPerTile], double (&sr)[kSubsPerTile]) {
  constexpr int stride = bwd_stride(S);
  const int lane = threadIdx.x & 63, ri = lane & 15, g = lane >> 4;
#pragma unroll 1
  for (int k0 = kb; k0 < ke; k0 += 64) {
    const int m = min(64, ke - k0);
    const int vidx = lane < m ? (int)lst[k0 + lane] : 0;
#pragma unroll 1
    for (int q = 0; q < m; ++q) {
      const uint32_t e = (uint32_t)__builtin_amdgcn_readlane(vidx, q);
      const unsigned mask = entry_mask(e);
#pragma unroll
      for (int h = 0; h < kChunk / 16; ++h) {
        const int j0 = entry_chunk(e) * kChunk + h * 16;
        float qf[S];
        bwd_load<S>(qf, Q + bwd_at(j0 + ri, g, stride));
        const bwd_f4 xj = *reinterpret_cast<const bwd_f4*>(&T.xs[j0 + 4 * g]);
        const bwd_f4 yj = *reinterpret_cast<const bwd_f4*>(&T.ys[j0 + 4 * g]);
        double X[4], Y[4], R[4];
        if (!kWide) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            X[v] = (double)xj[v] - cx;
            Y[v] = (double)yj[v] - cy;
            R[v] = fma(X[v], X[v], Y[v] * Y[v]);
          }
        }
#pragma unroll
        for (int t = 0; t < kSubsPerTile; ++t) {
          if (!((mask >> t) & 1u)) continue;
          bwd_f4 sd = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s = 0; s < S; ++s) sd = __builtin_amdgcn_mfma_f32_16x16x4f32(qf[s], pf[t][s], sd, 0, 0, 0);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float dx = xi[t] - xj[v], dy = yi[t] - yj[v];
            const float d2 = fmaf(dx, dx, dy * dy);
            const double kt = (double)(exp2_fast(-(d2 * s2)) * sd[v]);
            s0[t] += kt;
            if (kWide) {
              const double DX = dx, DY = dy;
              sx[t] = fma(kt, DX, sx[t]);
              sy[t] = fma(kt, DY, sy[t]);
              sr[t] = fma(kt, fma(DX, DX, DY * DY), sr[t]);
            } else {
              sx[t] = fma(kt, X[v], sx[t]);
              sy[t] = fma(kt, Y[v], sy[t]);
              sr[t] = fma(kt, R[v], sr[t]);
            }
          }
        }
      }
    }
  }
}

// One wave's share of the plan (as the product's waves): per row tile it touches,
// part[slot][kBwdSums][64 rows].
template <int S>
__global__ __launch_bounds__(256, 3) void mvm_bwd_kernel(const TilePlan T, float s2, const float* __restrict__ P,
                                                         const float* __restrict__ Q, double* __restrict__ part) {
  const int w = plan_block(blockIdx.x, T.nw, T.wround) * kPlanWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int4 dsc = T.wdesc[w];
  int rest = T.wrest[w];
  if (dsc.x < 0) return;
  constexpr int stride = bwd_stride(S);
  const int lane = threadIdx.x & 63, ri = lane & 15, g = lane >> 4;
  int r = dsc.x, slot = dsc.y, kb = dsc.z, ke = dsc.w;
#pragma unroll 1
  while (true) {
    float xi[kSubsPerTile], yi[kSubsPerTile], pf[kSubsPerTile][S];
#pragma unroll
    for (int t = 0; t < kSubsPerTile; ++t) {
      const int i = r * kRowTile + t * kSubTile + ri;
      xi[t] = T.xs[i];
      yi[t] = T.ys[i];
      bwd_load<S>(pf[t], P + bwd_at(i, g, stride));
    }
    const float4 q0 = T.cbox[kChunksPerTile * r], q1 = T.cbox[kChunksPerTile * r + 1];
    const double ex = (double)fmaxf(q0.y, q1.y) - fminf(q0.x, q1.x), ey = (double)fmaxf(q0.w, q1.w) - fminf(q0.z, q1.z);
    const bool wide = __builtin_amdgcn_readfirstlane(fma(ex, ex, ey * ey) * s2 <= kWideTile ? 0 : 1);
    const double cx = wide ? 0.0 : (double)T.xs[r * kRowTile], cy = wide ? 0.0 : (double)T.ys[r * kRowTile];
    double s0[kSubsPerTile] = {}, sx[kSubsPerTile] = {}, sy[kSubsPerTile] = {}, sr[kSubsPerTile] = {};
    const uint32_t* lst = T.list + (size_t)r * T.nch;
    if (wide) bwd_accumulate<S, true>(T, s2, Q, lst, kb, ke, xi, yi, pf, cx, cy, s0, sx, sy, sr);
    else bwd_accumulate<S, false>(T, s2, Q, lst, kb, ke, xi, yi, pf, cx, cy, s0, sx, sy, sr);
    // over the four lane groups; lane 16 t + ri then ends row 16 t + ri
    double m0 = 0.0, mx = 0.0, my = 0.0, mr = 0.0;
    auto fold = [](double v) {
      v += __shfl_xor(v, 16, 64);
      return v + __shfl_xor(v, 32, 64);
    };
#pragma unroll
    for (int t = 0; t < kSubsPerTile; ++t) {
      const double a = fold(s0[t]), b = fold(sx[t]), c = fold(sy[t]), d = fold(sr[t]);
      if (g == t) m0 = a, mx = b, my = c, mr = d;
    }
    float xo = xi[0], yo = yi[0];
#pragma unroll
    for (int t = 1; t < kSubsPerTile; ++t)
      if (g == t) xo = xi[t], yo = yi[t];
    const double x = (double)xo - cx, y = (double)yo - cy;
    double* out = part + (size_t)slot * kBwdSums * kRowTile + lane;
    out[0] = wide ? mx : x * m0 - mx;
    out[kRowTile] = wide ? my : y * m0 - my;
    out[2 * kRowTile] = wide ? mr : fma(fma(x, x, y * y), m0, mr) - 2.0 * fma(x, mx, y * my);
    out[3 * kRowTile] = m0;
    if (rest <= 0) break;
    ++r;
    ++slot;
    kb = 0;
    ke = min(rest, T.count[r]);
    rest -= ke;
  }
}

// Sums of every row over its partial slots in order (and, gacc, over the passes);
// the last pass ends them: gpx[perm[i]] = -(a^2/l^2) sum, added to what is there with
// `add`, same for y. Per workgroup, part_h = the sums of K s d^2 and K s of its rows.
__global__ __launch_bounds__(256) void bwd_rows_kernel(const TilePlan T, const double* __restrict__ part, int first,
                                                       int last, int add, double scale, double* __restrict__ gacc,
                                                       float* gpx, float* gpy, double* __restrict__ part_h) {
  __shared__ double red[4];
  const int j = blockIdx.x * 256 + threadIdx.x, r = j / kRowTile, row = j % kRowTile;
  double v[kBwdSums] = {};
  if (r < T.nrt) {
    const int2 sl = T.rslot[r];
    const double* p = part + (size_t)sl.x * kBwdSums * kRowTile + row;
    for (int q0 = 0; q0 < sl.y; q0 += 4) {
      double t[4][kBwdSums];  // past the last slot the loads repeat it and are not added
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int k = 0; k < kBwdSums; ++k) t[u][k] = p[((size_t)min(q0 + u, sl.y - 1) * kBwdSums + k) * kRowTile];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (q0 + u < sl.y)
#pragma unroll
          for (int k = 0; k < kBwdSums; ++k) v[k] += t[u][k];
    }
  }
  const double sl = block_sum_double(v[2], red);
  if (threadIdx.x == 0) part_h[2 * blockIdx.x + 0] = sl;
  const double sf = block_sum_double(v[3], red);
  if (threadIdx.x == 0) part_h[2 * blockIdx.x + 1] = sf;
  if (j >= T.n) return;
  if (!first) {
    v[0] += gacc[2 * (size_t)j];
    v[1] += gacc[2 * (size_t)j + 1];
  }
  if (last) {
    const int dst = T.perm[j];
    const float x = (float)(scale * v[0]), y = (float)(scale * v[1]);
    gpx[dst] = add ? gpx[dst] + x : x;
    gpy[dst] = add ? gpy[dst] + y : y;
  } else {
    gacc[2 * (size_t)j] = v[0];
    gacc[2 * (size_t)j + 1] = v[1];
  }
}

// g_hyp[0] = (a^2/2) sum K s d^2 / l^3, g_hyp[1] = a sum K s (K without its a^2; one
// workgroup of 256 threads, each summing a fixed stride of the blocks, then a
// fixed tree).
__global__ __launch_bounds__(256) void bwd_reduce_hyp_kernel(int nblocks_total, const double* part_h, double l,
                                                             double a, double* g_hyp) {
  __shared__ double red[4];
  double sl = 0.0, sf = 0.0;
  for (int b = threadIdx.x; b < nblocks_total; b += blockDim.x) {
    sl += part_h[2 * b + 0];
    sf += part_h[2 * b + 1];
  }
  sl = block_sum_double(sl, red);
  sf = block_sum_double(sf, red);
  if (threadIdx.x == 0) {
    g_hyp[0] = 0.5 * a * a * sl / (l * l * l);
    g_hyp[1] = a * sf;
  }
}

struct BwdBufs {
  float *P, *Q;  // entries of one pass in the plan's order
  double *part, *gacc, *part_h;
};

static int bwd_passes(int npairs) { return cdiv(npairs, kMaxPass); }

template <class Cv>
static void carve_bwd(Cv& cv, int n, int npairs, BwdBufs& b) {
  const int npad = cdiv(n, kRowTile) * kRowTile;
  const size_t entries = (size_t)npad * 4 * bwd_stride(bwd_steps(std::min(npairs, kMaxPass)));
  b.P = cv.template take<float>(entries);
  b.Q = cv.template take<float>(entries);
  b.part = cv.template take<double>((size_t)plan_slots(n) * kBwdSums * kRowTile);
  b.gacc = cv.template take<double>(npairs > kMaxPass ? 2 * (size_t)npad : 1);
  b.part_h = cv.template take<double>((size_t)bwd_passes(npairs) * 2 * cdiv(npad, 256));
}

template <int S>
static int launch_bwd(const TilePlan& plan, const BwdBufs& b, float s2, int nc, int c0, const float* A, int lda,
                      const float* Bv, int ldb, const WChunk& w, hipStream_t stream) {
  hipLaunchKernelGGL(bwd_gather_kernel<S>, dim3(cdiv(4 * plan.npad, 256)), dim3(256), 0, stream, plan.n,
                     plan.npad, nc, c0, plan.perm, A, lda, Bv, ldb, w, b.P, b.Q);
  GPL_LAUNCH_CHECK();
  hipLaunchKernelGGL(mvm_bwd_kernel<S>, dim3(plan.nw / kPlanWaves), dim3(256), 0, stream, plan, s2, b.P, b.Q,
                     b.part);
  GPL_LAUNCH_CHECK();
  return GPL_OK;
}

// Gradient sums over a plan that holds every pair to be evaluated.
static int bwd_run(const TilePlan& plan, const BwdBufs& b, const gpl_kernel* kern, int npairs, const float* A, int lda,
                   const float* Bv, int ldb, const double* w, bool add, float* gpx, float* gpy, double* g_hyp,
                   hipStream_t stream) {
  const float s2 = (float)kernel_scale2(kern->lengthscale);
  const int blocks = cdiv(plan.npad, 256), passes = bwd_passes(npairs);
  const double scale = -(kern->amplitude * kern->amplitude) / (kern->lengthscale * kern->lengthscale);
  for (int pass = 0; pass < passes; ++pass) {
    const int c0 = pass * kMaxPass, nc = std::min(kMaxPass, npairs - c0), S = bwd_steps(nc);
    WChunk wd;
    for (int c = 0; c < kMaxPass; ++c) wd.w[c] = c >= nc ? 0.f : w ? (float)w[c0 + c] : 1.f;
    switch (S) {
      case 9: GPL_TRY((launch_bwd<9>(plan, b, s2, nc, c0, A, lda, Bv, ldb, wd, stream))); break;
      case 8: GPL_TRY((launch_bwd<8>(plan, b, s2, nc, c0, A, lda, Bv, ldb, wd, stream))); break;
      case 4: GPL_TRY((launch_bwd<4>(plan, b, s2, nc, c0, A, lda, Bv, ldb, wd, stream))); break;
      case 2: GPL_TRY((launch_bwd<2>(plan, b, s2, nc, c0, A, lda, Bv, ldb, wd, stream))); break;
      default: GPL_TRY((launch_bwd<1>(plan, b, s2, nc, c0, A, lda, Bv, ldb, wd, stream))); break;
    }
    hipLaunchKernelGGL(bwd_rows_kernel, dim3(blocks), dim3(256), 0, stream, plan, b.part, pass == 0 ? 1 : 0,
                       pass + 1 == passes ? 1 : 0, add ? 1 : 0, scale, b.gacc, gpx, gpy,
                       b.part_h + (size_t)pass * 2 * blocks);
    GPL_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(bwd_reduce_hyp_kernel, dim3(1), dim3(256), 0, stream, passes * blocks, b.part_h,
                     kern->lengthscale, kern->amplitude, g_hyp);
  GPL_LAUNCH_CHECK();
  return GPL_OK;
}

static size_t bwd_workspace(int n, int npairs) {
  Sizer s;
  BwdBufs b;
  carve_bwd(s, n, npairs, b);
  return s.used;
}

}  // namespace gpl

using namespace gpl;

extern "C" size_t gpl_gp_kernel_mvm_backward_workspace(int n, int npairs) {
  if (n <= 0 || npairs <= 0) return 0;
  Sizer s;
  TilePlan plan;
  BwdBufs b;
  plan_carve(s, n, plan);
  carve_bwd(s, n, npairs, b);
  return s.used;
}

static int check_backward(const gpl_kernel* kern, int n, int npairs) {
  GPL_TRY(check_kernel(kern));
  GPL_REQUIRE(n >= 1 && npairs >= 1 && npairs <= 4096, "n=%d npairs=%d out of range", n, npairs);
  GPL_REQUIRE(kern->amplitude != 0.0, "amplitude must be non-zero for the amplitude gradient");
  return GPL_OK;
}

extern "C" int gpl_gp_kernel_mvm_backward(const gpl_kernel* kern, int n, const float* px, const float* py,
                                          int npairs, const float* A, int lda, const float* Bv, int ldb,
                                          const double* w, float* gpx, float* gpy, double* g_hyp, void* ws,
                                          size_t ws_bytes, hipStream_t stream) {
  GPL_TRY(check_backward(kern, n, npairs));
  GPL_REQUIRE(px && py && A && Bv && w && gpx && gpy && g_hyp, "NULL argument");
  GPL_REQUIRE(lda >= n && ldb >= n, "lda/ldb must be >= n");
  for (int c = 0; c < npairs; ++c) GPL_REQUIRE(std::isfinite(w[c]), "weight %d is not finite", c);
  GPL_TRY(check_ws(ws, ws_bytes, gpl_gp_kernel_mvm_backward_workspace(n, npairs)));
  Carver cv(ws, ws_bytes);
  TilePlan plan;
  BwdBufs b;
  plan_carve(cv, n, plan);
  carve_bwd(cv, n, npairs, b);
  if (!cv.ok()) return check_ws(nullptr, 0, 1);
  const float s2 = (float)kernel_scale2(kern->lengthscale);
  GPL_TRY(plan_build(plan, n, px, py, nullptr, s2, kSkipBackward, kSkipBackward, stream));
  return bwd_run(plan, b, kern, npairs, A, lda, Bv, ldb, w, true, gpx, gpy, g_hyp, stream);
}

// The plan of the product serves its adjoint too: both keep the pairs below the same
// threshold (kSkipBackward), and the precision form's mask of pairs that need the lo part
// changes the plan's split of the work, not the pairs.
static_assert(kSkipBackward == kSkipFp32 && kSkipBackward == kSkipF16x3, "one plan for both");

extern "C" size_t gpl_gp_kernel_mvm_vjp_workspace(int n, int ncols, int prec) {
  if (n <= 0 || ncols <= 0 || ncols > 4096) return 0;
  return align_up(mvm_workspace(n, ncols, prec)) + bwd_workspace(n, ncols) + kAlign;
}

extern "C" int gpl_gp_kernel_mvm_vjp(const gpl_kernel* kern, int n, const float* px, const float* py, int ncols,
                                     const float* V, int ldv, const float* G, int ldg, float* gV, int ldgv, float* gpx,
                                     float* gpy, double* g_hyp, int prec, void* ws, size_t ws_bytes,
                                     hipStream_t stream) {
  GPL_TRY(check_backward(kern, n, ncols));
  GPL_REQUIRE(prec == GPL_PREC_FP32 || prec == GPL_PREC_F16X3, "unknown precision %d", prec);
  GPL_REQUIRE(px && py && V && G && gV && gpx && gpy && g_hyp, "NULL argument");
  GPL_REQUIRE(ldv >= n && ldg >= n && ldgv >= n, "ldv/ldg/ldgv must be >= n");
  GPL_REQUIRE(V != gV && G != gV, "gV must not overlap its operands");
  GPL_TRY(check_ws(ws, ws_bytes, gpl_gp_kernel_mvm_vjp_workspace(n, ncols, prec)));
  Carver cv(ws, ws_bytes);
  const size_t mb = mvm_workspace(n, ncols, prec);
  char* mws = cv.take<char>(mb);
  BwdBufs b;
  carve_bwd(cv, n, ncols, b);
  if (!cv.ok()) return check_ws(nullptr, 0, 1);
  MvmCtx m;
  GPL_TRY(mvm_prepare(m, kern->lengthscale, kern->amplitude, n, px, py, nullptr, ncols, prec, false, mws, mb, stream,
                      G, ldg));
  GPL_TRY(mvm_run_prepared(m, ncols, gV, ldgv, 0.f, CgGate{}, stream, true));  // K is symmetric
  return bwd_run(m.plan, b, kern, ncols, G, ldg, V, ldv, nullptr, false, gpx, gpy, g_hyp, stream);
}
