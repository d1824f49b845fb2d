// Variationally optimised GP source: one reparametrised ELBO sample and its
// gradient (Sec. 3.3 eqs. "gp-gen2", "decomposition"; Sec. 3.4 eq.
// "transmission" with the k-th-neighbour density; Sec. 3.5 image- and
// source-plane layers; Sec. 3.6 eqs. "elbo", "reparam"; Sec. 4.2 eq. "guide"),
// and the Adam update of Sec. 4.3.
//
// Layers: f = mu(p) + sum_k T_k y_k, T_k[i][j] = A_j N(p_i - q_j, Zt_i + l_k^2 I / 2),
// A_j = sqrt(2 pi l_k^2) w_j with w_j = rho_j^{-1/2} = r_j sqrt(pi / k) (r_j the
// distance to the k-th closest other inducing point). Image-plane layers: q = p,
// Zt = the pixel shapes; the source-plane layer: q = a fixed grid, Zt = 0. All
// products are the Gaussian products of gauss_tiles.hip over the points sorted
// once per step (every pair that is not exactly zero in FP32).
//
// Step: the lens sample theta (device FP64), the source samples y (FP32),
// ray tracing from the device-held theta, pixel shapes, k-NN weights, the
// layered fluxes, residual r = d - B f; backward g_f = B^T r / sigma^2, per
// layer T_k^T g_f, then dE/dp from the Sersic mean, both sides of every
// transmission product, the pixel shapes and the k-NN weights, and dE/dtheta
// by the ray-tracing adjoint. A final one-workgroup kernel folds the FP64 sums
// into the ELBO pieces and the gradient of the small FP64 parameter block.
//
// A launch takes some 4.6 us in such a chain whatever it does, so the work of the
// small steps is joined: every layer's launches are one, clears and per-point steps
// ride on a launch that touches the same points, and partial sums are folded where
// they are used: 23 launches for 57, 853 -> 579 us a step at 40,000 traced points, three
// layers and a 40 x 40 grid, 18 for 44 and 222 -> 149 us at 4,096 points (480 and 138
// with what the products and the sorts have gained since).
//
// Each layer takes two passes over its pairs, not four. The adjoint of T_k y
// towards the targets is g_f[i] times sums over j of the same terms as the
// product itself (G_ij A_j y_j times 1, C_i^{-1} d and its products), so the
// forward pass forms them too; the adjoint towards the inducing points is y_j
// times sums over i of the terms of T_k^T g_f (G_ij g_f[i] times 1 and C_i^{-1} d),
// formed together with it.
#include <cmath>

#include "common.hpp"
#include "gauss_tiles.hpp"
#include "internal.hpp"
#include "pixel_axes.hpp"
#include "sersic.hpp"

namespace gpl {

constexpr int kVMaxLayers = 8;
static_assert(kVMaxLayers <= kGaussLayers, "one launch for all layers");
constexpr int kVSums = 1 + 3 * kVMaxLayers;  // |r|^2, then per layer |y|^2, sum log s, |e|^2
constexpr int kVSumParts = 32;               // workgroups of each sum

struct VLayout {
  int nl, nip, sp;  // layers, image-plane layers, index of the source-plane layer (-1: none)
  int N, M, G, npix;
  size_t n64, n32, ne32;
  size_t mean[kVMaxLayers], logs[kVMaxLayers], cross;  // P32 offsets of each layer's blocks
  size_t e[kVMaxLayers];                               // e32 offset of each layer's noise
  int n[kVMaxLayers];                                  // source parameters per layer
};

static int vigp_layout(const gpl_vigp_model* m, const gpl_grid* grid, int G, VLayout& L) {
  GPL_REQUIRE(m != nullptr && grid != nullptr, "model/grid are NULL");
  GPL_REQUIRE(m->n_layers >= 1 && m->n_layers <= kVMaxLayers, "n_layers=%d must be in [1, %d]", m->n_layers,
              kVMaxLayers);
  GPL_REQUIRE(grid->n >= 1 && grid->ss >= 1, "bad grid");
  L.nl = m->n_layers;
  L.M = grid->n * grid->ss;
  L.N = L.M * L.M;
  L.npix = grid->n * grid->n;
  L.G = G;
  L.sp = -1;
  L.nip = 0;
  for (int k = 0; k < L.nl; ++k) {
    GPL_REQUIRE(m->lengthscale[k] > 0 && std::isfinite(m->lengthscale[k]), "lengthscale[%d] must be > 0", k);
    if (m->kind[k] == GPL_VIGP_SOURCE_PLANE) {
      GPL_REQUIRE(L.sp < 0, "at most one source-plane layer");
      L.sp = k;
    } else {
      GPL_REQUIRE(m->kind[k] == GPL_VIGP_IMAGE_PLANE, "kind[%d]=%d unknown", k, m->kind[k]);
      ++L.nip;
    }
  }
  GPL_REQUIRE(m->knn_k >= 1 && m->knn_k <= 32, "knn_k=%d must be in [1, 32]", m->knn_k);
  GPL_REQUIRE(L.nip == 0 || L.N > m->knn_k, "need more than knn_k traced points");
  GPL_REQUIRE(L.sp < 0 || G > m->knn_k, "a source-plane layer needs more than knn_k grid points (G=%d)", G);
  GPL_REQUIRE(m->shear_sd > 0, "shear_sd must be > 0");
  L.n64 = 56 + (size_t)L.nl;
  size_t o = 0, oe = 0;
  if (L.sp >= 0) {
    L.mean[L.sp] = o;
    L.logs[L.sp] = o + G;
    L.cross = o + 2 * (size_t)G;
    L.n[L.sp] = G;
    L.e[L.sp] = oe;
    o += 9 * (size_t)G;
    oe += G;
  }
  for (int k = 0; k < L.nl; ++k) {
    if (k == L.sp) continue;
    L.mean[k] = o;
    L.logs[k] = o + L.N;
    L.n[k] = L.N;
    L.e[k] = oe;
    o += 2 * (size_t)L.N;
    oe += L.N;
  }
  L.n32 = o;
  L.ne32 = oe;
  return GPL_OK;
}

// bump allocation inside the caller's workspace
struct Bump {
  char* p;
  size_t used = 0;
  template <class T>
  T* take(size_t n) {
    T* r = p ? reinterpret_cast<T*>(p + used) : nullptr;
    used += align_up(n * sizeof(T));
    return r;
  }
};

struct VBufs {
  double *lens, *sums, *gq, *rt_partial;
  TilePlan sort_p, sort_g;  // the traced points and the source-plane grid along the curve
  char* tiles;
  size_t tiles_bytes;
  float *px, *py, *Z, *f, *resid, *g_f, *gpx, *gpy, *gZ, *r, *w, *w_sp, *y;
  float* tg;  // [5][N] adjoint towards the targets per unit of g_f: dx, dy, shape xx, xy, yy
  int* nn;
  int* far_count;  // [kVMaxLayers] targets of each layer whose shapes reach far
};

static size_t vigp_carve(const VLayout& L, void* ws, VBufs& b) {
  Bump B{static_cast<char*>(ws)};
  const size_t N = L.N, G = std::max(L.G, 1);
  b.lens = B.take<double>(8);
  b.sums = B.take<double>(kVSums * kVSumParts);
  b.gq = B.take<double>(2 * N);
  b.rt_partial = B.take<double>(8 * (size_t)cdiv(L.N, 256));
  b.px = B.take<float>(N);
  b.py = B.take<float>(N);
  b.Z = B.take<float>(3 * N);
  b.f = B.take<float>(N);
  b.resid = B.take<float>(L.npix);
  b.g_f = B.take<float>(N);
  b.gpx = B.take<float>(N);
  b.gpy = B.take<float>(N);
  b.gZ = B.take<float>(3 * N);
  b.r = B.take<float>(N);
  b.w = B.take<float>(N);
  b.nn = B.take<int>(N);
  b.w_sp = B.take<float>(G);
  b.y = B.take<float>(L.ne32 ? L.ne32 : 1);
  b.tg = B.take<float>(5 * N);
  b.far_count = B.take<int>(kVMaxLayers);
  sort_carve(B, L.N, b.sort_p);
  if (L.sp >= 0) sort_carve(B, L.G, b.sort_g);
  b.tiles_bytes = std::max(gauss_layers_scratch(L.n, L.N, L.nl), gauss_ordered_scratch(L.N, L.n, L.nl));
  b.tiles = B.take<char>(b.tiles_bytes);
  return B.used;
}

struct VSeg {
  const float* a[kVSums];
  int n[kVSums];
  int square[kVSums];
};

// sums[s][q] = the q-th of kVSumParts strided parts of sum_i a_s[i]^2 (square) or
// sum_i a_s[i], FP64 in a fixed order.
__global__ __launch_bounds__(256) void vigp_sums_kernel(VSeg seg, double* sums) {
  __shared__ double red[4];
  const int s = blockIdx.y;
  const float* a = seg.a[s];
  const int n = seg.n[s];
  double acc = 0.0;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += 256 * kVSumParts) {
    const double v = (double)a[i];
    acc += seg.square[s] ? v * v : v;
  }
  acc = block_sum_double(acc, red);
  if (threadIdx.x == 0) sums[s * kVSumParts + blockIdx.x] = acc;
}

struct VSample {
  int sp, ne, ngq;
  int e[kVMaxLayers], n[kVMaxLayers];  // noise offset and size of each layer
  const float *m[kVMaxLayers], *logs[kVMaxLayers], *cross;
};

// The samples. Of the source parameters, y = m + C e_l + exp(logs) e (C, n x 7 with
// column b at b n, for the source-plane layer only). The last workgroup: the lens,
// theta = m_l + L_l e_l (L_l: strictly lower part of raw, exp of its diagonal), with the
// fixed slope in position 3 of the 8-vector. Also clears gq and the layers' counts.
__global__ __launch_bounds__(256) void vigp_sample_kernel(VSample S, const double* __restrict__ P64,
                                                          const double* __restrict__ e_l,
                                                          const float* __restrict__ e, double slope, double* lens,
                                                          float* __restrict__ y, double* __restrict__ gq,
                                                          int* far_count) {
  if (blockIdx.x + 1 == gridDim.x) {
    const int a = threadIdx.x;
    if (a < kVMaxLayers) far_count[a] = 0;
    if (a < 7) {
      double t = P64[a];
      for (int b = 0; b < a; ++b) t += P64[7 + a * 7 + b] * e_l[b];
      t += exp(P64[7 + a * 7 + a]) * e_l[a];
      lens[a < 3 ? a : a + 1] = t;
    }
    if (a == 7) lens[3] = slope;
    return;
  }
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < S.ngq) gq[i] = 0.0;
  if (i >= S.ne) return;
  int k = 0;
  while (i < S.e[k] || i >= S.e[k] + S.n[k]) ++k;  // the layers cover [0, ne)
  const int j = i - S.e[k], n = S.n[k];
  float v = S.m[k][j];
  if (k == S.sp)
    for (int b = 0; b < 7; ++b) v = fmaf(S.cross[(size_t)b * n + j], (float)e_l[b], v);
  y[i] = fmaf(expf(S.logs[k][j]), e[i], v);
}

// Per traced point: its pixel shape and the mean function, f = mu(p).
__global__ __launch_bounds__(256) void vigp_points_kernel(int M, SersicF S, const float* __restrict__ px,
                                                          const float* __restrict__ py, float* Z, float* f) {
  const int j = blockIdx.x * 256 + threadIdx.x, N = M * M;
  if (j >= N) return;
  store_shape(pixel_axes(M, j, px, py), N, j, Z);
  float t;
  f[j] = sersic_shape(S, px[j] - S.xs, py[j] - S.ys, t);
}

struct VLayerAdj {
  const float *part, *w, *y, *logs, *e;
  const double* log_amp;
  float *gmean, *glogs;
  float norm;
  int nslices;
};
struct VAdj {
  int nip;
  VLayerAdj ip[kVMaxLayers], sp;
  GSorted P, Q;
  float* gcross;
  // image-plane points: distance to and index of the k-th neighbour, positions
  const float *r, *px, *py;
  const int* nn;
  float *gpx, *gpy;
  double* gq;
};

// Inducing point j of a layer: t_j = (T^T g_f)_j = norm w_j sum, and the parameter
// gradients g_y = t - y / alpha^2 (alpha = exp(log_amp)); dE/dm = g_y, dE/dlog s =
// s g_y e + 1. Returns g_y.
__device__ __forceinline__ float adjoint_point(const VLayerAdj& L, int j, float wj, float s, float yj) {
  const float ia2 = (float)exp(-2.0 * L.log_amp[0]);
  const float g = L.norm * wj * s - yj * ia2;
  L.gmean[j] = g;
  L.glogs[j] = fmaf(expf(L.logs[j]) * g, L.e[j], 1.f);
  return g;
}

// End of the transposed passes. blockIdx.y 0: the traced points, sorted point i, over
// the image-plane layers; these add the adjoint towards the inducing points, norm y_j w_j
// sum G C^{-1} (t - q) to their positions (the sums hold kFormScale C^{-1} (q - t)), and
// norm y_j sum G to the weights. Weights w_j = r_j sqrt(pi / k) (rho^{-1/2}, rho = k /
// (pi r^2)), r_j = |q_j - q_nn(j)|: dF/dq_j += coef v, dF/dq_nn(j) -= coef v with
// v = q_j - q_nn(j), coef = gw_j w_j / r_j^2; both shares are scattered with FP64 atomic
// adds into gq (2n doubles: x then y), so that a point's shares, which may cancel, are
// rounded to FP32 once, as their sum (its own rounded by itself saves 1 us a step).
// blockIdx.y 1: the source-plane layer, dE/dC[:, b] = g_y e_l[b].
__global__ __launch_bounds__(256) void vigp_adjoint_kernel(VAdj A, const double* __restrict__ e_l) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (blockIdx.y == 1) {
    const VLayerAdj& L = A.sp;
    const int n = A.Q.n;
    if (i >= n) return;
    const int j = A.Q.perm[i];
    const float g = adjoint_point(L, j, L.w[j], fold_slices(L.part, L.nslices, 1, A.Q.nch * kChunk, 0, i), L.y[j]);
    for (int b = 0; b < 7; ++b) A.gcross[(size_t)b * n + j] = g * (float)e_l[b];
    return;
  }
  const int n = A.P.n;
  if (i >= n || A.nip == 0) return;
  const int j = A.P.perm[i], npt = A.P.nch * kChunk;
  const float wj = A.ip[0].w[j];  // the layers share the weights
  float gx = A.gpx[j], gy = A.gpy[j], gw = 0.f;
  for (int k = 0; k < A.nip; ++k) {
    const VLayerAdj& L = A.ip[k];
    float s[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) s[q] = fold_slices(L.part, L.nslices, 3, npt, q, i);
    const float yj = L.y[j];
    adjoint_point(L, j, wj, s[0], yj);
    const float c = -L.norm * yj * wj / kFormScale;
    gx += c * s[1];
    gy += c * s[2];
    gw += L.norm * yj * s[0];
  }
  const int o = A.nn[j];
  const float r = A.r[j];
  if (o >= 0 && r > 0.f) {
    const double coef = (double)gw * (double)wj / ((double)r * (double)r);
    const double vx = coef * (double)(A.px[j] - A.px[o]), vy = coef * (double)(A.py[j] - A.py[o]);
    atomicAdd(A.gq + j, vx);
    atomicAdd(A.gq + n + j, vy);
    atomicAdd(A.gq + o, -vx);
    atomicAdd(A.gq + n + o, -vy);
  }
  A.gpx[j] = gx;
  A.gpy[j] = gy;
}

// dE/dp by the mean function and the targets' side of the layers (g_f times the sums
// of the forward passes), and with shapes dE/dZ.
__global__ void vigp_target_kernel(int N, int shapes, SersicF S, const float* __restrict__ px,
                                   const float* __restrict__ py, const float* __restrict__ g_f,
                                   const float* __restrict__ tg, float* gpx, float* gpy, float* gZ) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const float g = g_f[i], dx = px[i] - S.xs, dy = py[i] - S.ys, m = sersic_slope(S, dx, dy);
  gpx[i] = g * fmaf(m, dx, tg[i]);
  gpy[i] = g * fmaf(m, dy, tg[N + i]);
  if (shapes)
#pragma unroll
    for (int k = 0; k < 3; ++k) gZ[(size_t)k * N + i] = g * tg[(size_t)(2 + k) * N + i];
}

struct VFinal {
  int nl, n[kVMaxLayers], nparts;
  double half_inv_var, lo[5], hi[5], inv_shear_var;
  double loglik0, lpy0[kVMaxLayers], lpt0, nlq0;  // the terms that depend on the model alone
};

// ELBO pieces and the FP64 gradient block (lens mean 7, lens raw 49, log amp). Wave k
// folds the partial sums of lens parameter k, then every eighth segment's; thread
// a < 49 writes entry a of the lens block's raw part.
__global__ __launch_bounds__(512) void vigp_finalize_kernel(VFinal F, const double* __restrict__ P64,
                                                            const double* __restrict__ e_l,
                                                            const double* __restrict__ lens,
                                                            const double* __restrict__ parts,
                                                            const double* __restrict__ rt, double* out, double* G64) {
  __shared__ double gt8[8], sums[kVSums];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  {
    double s = 0.0;
    for (int b = lane; b < F.nparts; b += 64) s += rt[(size_t)b * 8 + w];
    s = warp_sum(s);
    if (lane == 0) gt8[w] = w >= 6 ? s - lens[w] * F.inv_shear_var : s;
  }
  for (int k = w; k < 1 + 3 * F.nl; k += 8) {
    const double s = wave_fold_sum(parts + k * kVSumParts, kVSumParts);
    if (lane == 0) sums[k] = s;
  }
  __syncthreads();
  auto grad = [&](int a) { return gt8[a < 3 ? a : a + 1]; };
  if (tid < 49) {
    const int a = tid / 7, b = tid - 7 * a;
    const double g = grad(a);
    double v = 0.0;
    if (b < a) v = g * e_l[b];
    if (b == a) v = g * e_l[a] * exp(P64[7 + a * 7 + a]) + 1.0;
    G64[7 + tid] = v;
    if (b == 0) G64[a] = g;
  }
  if (tid < 8) out[5 + tid] = lens[tid];
  if (tid != 64) return;
  const double loglik = F.loglik0 - F.half_inv_var * sums[0];
  double lpy = 0.0, nlq = F.nlq0, lpt = F.lpt0;
  for (int a = 0; a < 7; ++a) nlq += 0.5 * e_l[a] * e_l[a] + P64[7 + a * 7 + a];
  for (int k = 0; k < F.nl; ++k) {
    const double la = P64[56 + k], sya2 = sums[1 + 3 * k] * exp(-2.0 * la);
    lpy += -0.5 * sya2 - F.n[k] * la + F.lpy0[k];
    nlq += 0.5 * sums[3 + 3 * k] + sums[2 + 3 * k];
    G64[56 + k] = sya2 - F.n[k];
  }
  bool inside = true;
  for (int i = 0; i < 5; ++i) {
    const double t = lens[i < 3 ? i : i + 1];
    inside = inside && t >= F.lo[i] && t <= F.hi[i];
  }
  if (!inside) lpt = -INFINITY;
  for (int k = 6; k < 8; ++k) lpt -= 0.5 * lens[k] * lens[k] * F.inv_shear_var;
  out[0] = loglik + lpy + lpt + nlq;
  out[1] = loglik;
  out[2] = lpy;
  out[3] = lpt;
  out[4] = nlq;
}

// Adam (torch's form) minimising -E: the loss gradient is -G. The weights
// 1 - beta come from the host in double precision (1 - 0.999f in FP32 would be
// 1.3e-5 off 0.001).
template <class T>
struct AdamBlock {
  size_t n;
  T* p;
  const T* g;
  T *m, *v;
  T lr_bc1, b1, omb1, b2, omb2, inv_sqrt_bc2, eps;
  __device__ __forceinline__ void update(size_t j) const {
    if (j >= n) return;
    const T gl = -g[j];
    const T mj = b1 * m[j] + omb1 * gl;
    const T vj = b2 * v[j] + omb2 * gl * gl;
    m[j] = mj;
    v[j] = vj;
    p[j] -= lr_bc1 * mj / (sqrt(vj) * inv_sqrt_bc2 + eps);
  }
};

// The first blocks64 workgroups update the FP64 block, the others the FP32 one.
__global__ __launch_bounds__(256) void vigp_adam_kernel(unsigned blocks64, AdamBlock<double> d, AdamBlock<float> s) {
  if (blockIdx.x < blocks64) d.update((size_t)blockIdx.x * 256 + threadIdx.x);
  else s.update((size_t)(blockIdx.x - blocks64) * 256 + threadIdx.x);
}

static inline dim3 blocks_for(size_t n) { return dim3((unsigned)((n + 255) / 256)); }

}  // namespace gpl

using namespace gpl;

extern "C" int gpl_vigp_sizes(const gpl_vigp_model* model, const gpl_grid* grid, int G, size_t* n64, size_t* n32,
                              size_t* ne32) {
  VLayout L;
  GPL_TRY(vigp_layout(model, grid, G, L));
  if (n64) *n64 = L.n64;
  if (n32) *n32 = L.n32;
  if (ne32) *ne32 = L.ne32;
  return GPL_OK;
}

extern "C" size_t gpl_vigp_workspace(const gpl_vigp_model* model, const gpl_grid* grid, int G) {
  VLayout L;
  if (vigp_layout(model, grid, G, L) != GPL_OK) return 0;
  VBufs b{};
  return vigp_carve(L, nullptr, b);
}

extern "C" int gpl_vigp_elbo(const gpl_vigp_model* model, const gpl_grid* grid, const gpl_psf* psf,
                             const gpl_source* src, double noise_sigma, int G, const float* gx, const float* gy,
                             const float* d, const double* P64, const float* P32, const double* e64,
                             const float* e32, double* out, double* G64, float* G32, void* ws, size_t ws_bytes,
                             hipStream_t stream) {
  VLayout L;
  GPL_TRY(vigp_layout(model, grid, G, L));
  GPL_REQUIRE(noise_sigma > 0 && std::isfinite(noise_sigma), "noise_sigma must be > 0");
  GPL_REQUIRE(src != nullptr && psf != nullptr, "source/psf are NULL");
  GPL_TRY(check_source(src));
  GPL_REQUIRE(d && P64 && P32 && e64 && e32 && out && G64 && G32, "NULL argument");
  GPL_REQUIRE(L.sp < 0 || (gx && gy), "source-plane layer without grid points");
  for (int i = 0; i < 5; ++i)
    GPL_REQUIRE(model->prior_hi[i] > model->prior_lo[i], "prior box %d is empty", i);
  VBufs b{};
  const size_t need = vigp_carve(L, nullptr, b);
  GPL_TRY(check_ws(ws, ws_bytes, need));
  vigp_carve(L, ws, b);
  const int N = L.N;
  const double kk = model->knn_k;
  const float wscale = (float)std::sqrt(M_PI / kk);

  const SersicF sersic = make_sersic(src);
  Taps taps;
  GPL_TRY(make_taps(grid, psf, taps));

  // ---- samples
  const float* y[kVMaxLayers];
  VSample smp{};
  smp.sp = L.sp;
  smp.ne = (int)L.ne32;
  smp.ngq = L.nip > 0 ? 2 * N : 0;
  if (L.sp >= 0) smp.cross = P32 + L.cross;
  for (int k = 0; k < L.nl; ++k) {
    y[k] = b.y + L.e[k];
    smp.e[k] = (int)L.e[k];
    smp.n[k] = L.n[k];
    smp.m[k] = P32 + L.mean[k];
    smp.logs[k] = P32 + L.logs[k];
  }
  hipLaunchKernelGGL(vigp_sample_kernel, dim3(cdiv(std::max(smp.ne, smp.ngq), 256) + 1), dim3(256), 0, stream, smp, P64,
                     e64, e32, model->slope, b.lens, b.y, b.gq, b.far_count);
  GPL_LAUNCH_CHECK();
  // ---- forward
  GPL_TRY(raytrace_dev_launch(grid, b.lens, b.px, b.py, stream));
  hipLaunchKernelGGL(vigp_points_kernel, blocks_for(N), dim3(256), 0, stream, L.M, sersic, b.px, b.py, b.Z, b.f);
  GPL_LAUNCH_CHECK();
  if (L.sp >= 0) GPL_TRY(plan_sort_pair(b.sort_p, N, b.px, b.py, b.sort_g, G, gx, gy, stream));
  else GPL_TRY(plan_sort(b.sort_p, N, b.px, b.py, stream));
  KnnSet sets[2];
  int nsets = 0;
  if (L.nip > 0) sets[nsets++] = KnnSet{b.sort_p, nullptr, b.r, b.w, b.nn};
  if (L.sp >= 0) sets[nsets++] = KnnSet{b.sort_g, nullptr, nullptr, b.w_sp, nullptr};
  GPL_TRY(knn_sorted_launch(sets, nsets, model->knn_k, wscale, stream));
  const GSorted P = sorted_view(b.sort_p), Q = sorted_view(b.sort_g);
  GaussLayer fwd[kVMaxLayers];
  GaussLayerSums adj[kVMaxLayers];
  for (int k = 0; k < L.nl; ++k) {
    const double ell = model->lengthscale[k], base = 0.5 * ell * ell;
    const bool sp = k == L.sp;
    fwd[k] = GaussLayer{sp ? GSide{gx, gy, nullptr, b.w_sp, G} : GSide{b.px, b.py, nullptr, b.w, N}, sp ? 0 : 1, base,
                        std::sqrt(2.0 * M_PI * ell * ell) / (2.0 * M_PI), y[k]};
    adj[k] = GaussLayerSums{sp ? Q : P, sp ? 0 : 1, base, nullptr, 0};
  }
  GPL_TRY(gauss_ordered_launch(P, b.Z, fwd, L.nl, b.f, b.tg, b.far_count, b.tiles, b.tiles_bytes, stream));
  GPL_TRY(psf_forward_launch(grid->n, grid->ss, taps, 1, b.f, N, b.resid, L.npix, -1.f, 0.f, d, L.npix, 1.f, nullptr, 0,
                             nullptr, CgGate{}, stream));  // r = d - B f
  // ---- backward
  GPL_TRY(psf_adjoint_launch(grid->n, grid->ss, taps, 1, b.resid, L.npix, b.g_f, N,
                             (float)(1.0 / (noise_sigma * noise_sigma)), 0.f, CgGate{},
                             stream));  // g_f = B^T r / sigma^2
  hipLaunchKernelGGL(vigp_target_kernel, blocks_for(N), dim3(256), 0, stream, N, L.nip > 0 ? 1 : 0, sersic, b.px, b.py,
                     b.g_f, b.tg, b.gpx, b.gpy, b.gZ);
  GPL_LAUNCH_CHECK();
  // T_k^T g_f: targets are the inducing points (weights A), sources the traced points
  GPL_TRY(gauss_layers_sums(adj, L.nl, P, b.Z, b.g_f, b.tiles, b.tiles_bytes, stream));
  VAdj A{};
  for (int k = 0; k < L.nl; ++k) {
    const bool sp = k == L.sp;
    const float base = (float)adj[k].base;
    const VLayerAdj q{adj[k].part, sp ? b.w_sp : b.w, y[k], P32 + L.logs[k], e32 + L.e[k], P64 + 56 + k,
                      G32 + L.mean[k], G32 + L.logs[k],
                      sp ? (float)fwd[k].norm / std::sqrt(base * base) : (float)fwd[k].norm, adj[k].nslices};
    if (sp) A.sp = q;
    else A.ip[A.nip++] = q;
  }
  A.P = P;
  A.Q = Q;
  A.gcross = L.sp >= 0 ? G32 + L.cross : nullptr;
  A.r = b.r;
  A.px = b.px;
  A.py = b.py;
  A.nn = b.nn;
  A.gpx = b.gpx;
  A.gpy = b.gpy;
  A.gq = b.gq;
  hipLaunchKernelGGL(vigp_adjoint_kernel, dim3(cdiv(std::max(N, L.sp >= 0 ? G : 0), 256), L.sp >= 0 ? 2 : 1), dim3(256),
                     0, stream, A, e64);
  GPL_LAUNCH_CHECK();
  const bool ip = L.nip > 0;
  GPL_TRY(raytrace_dev_backward_launch(
      grid, b.lens, PointGrads{b.gpx, b.gpy, ip ? b.gq : nullptr, ip ? b.gZ : nullptr, b.px, b.py}, b.rt_partial,
      stream));
  // ---- scalars
  VSeg seg{};
  int ns = 0;
  auto segment = [&](const float* a, int n, int square) {
    seg.a[ns] = a;
    seg.n[ns] = n;
    seg.square[ns++] = square;
  };
  segment(b.resid, L.npix, 1);
  for (int k = 0; k < L.nl; ++k) {
    segment(y[k], L.n[k], 1);
    segment(P32 + L.logs[k], L.n[k], 0);
    segment(e32 + L.e[k], L.n[k], 1);
  }
  hipLaunchKernelGGL(vigp_sums_kernel, dim3(kVSumParts, ns), dim3(256), 0, stream, seg, b.sums);
  GPL_LAUNCH_CHECK();
  const double l2pi = std::log(2.0 * M_PI);
  VFinal F{};
  F.nl = L.nl;
  F.nparts = cdiv(N, 256);
  F.half_inv_var = 0.5 / (noise_sigma * noise_sigma);
  F.loglik0 = -L.npix * std::log(noise_sigma) - 0.5 * L.npix * l2pi;
  double ntot = 7.0;
  for (int k = 0; k < L.nl; ++k) {
    F.n[k] = L.n[k];
    F.lpy0[k] = -0.5 * L.n[k] * l2pi;
    ntot += L.n[k];
  }
  F.nlq0 = 0.5 * ntot * l2pi;
  for (int i = 0; i < 5; ++i) {
    F.lo[i] = model->prior_lo[i];
    F.hi[i] = model->prior_hi[i];
    F.lpt0 -= std::log(F.hi[i] - F.lo[i]);
  }
  F.lpt0 -= 2.0 * std::log(model->shear_sd) + l2pi;
  F.inv_shear_var = 1.0 / (model->shear_sd * model->shear_sd);
  hipLaunchKernelGGL(vigp_finalize_kernel, dim3(1), dim3(512), 0, stream, F, P64, e64, b.lens, b.sums, b.rt_partial, out,
                     G64);
  GPL_LAUNCH_CHECK();
  return GPL_OK;
}

extern "C" int gpl_vigp_adam(size_t n64, double* P64, const double* G64, double* M64, double* V64, size_t n32,
                             float* P32, const float* G32, float* M32, float* V32, int t, double lr, double beta1,
                             double beta2, double eps, hipStream_t stream) {
  GPL_REQUIRE(t >= 1, "step t=%d must be >= 1", t);
  GPL_REQUIRE(lr > 0 && beta1 >= 0 && beta1 < 1 && beta2 >= 0 && beta2 < 1 && eps > 0, "bad Adam constants");
  const double bc1 = 1.0 - std::pow(beta1, t), bc2 = 1.0 - std::pow(beta2, t);
  GPL_REQUIRE(n64 == 0 || (P64 && G64 && M64 && V64), "NULL FP64 block");
  GPL_REQUIRE(n32 == 0 || (P32 && G32 && M32 && V32), "NULL FP32 block");
  if (n64 == 0 && n32 == 0) return GPL_OK;
  const double isb = 1.0 / std::sqrt(bc2);
  const AdamBlock<double> d{n64, P64, G64, M64, V64, lr / bc1, beta1, 1.0 - beta1, beta2, 1.0 - beta2, isb, eps};
  const AdamBlock<float> s{n32, P32, G32, M32, V32, (float)(lr / bc1), (float)beta1, (float)(1.0 - beta1),
                           (float)beta2, (float)(1.0 - beta2), (float)isb, (float)eps};
  const unsigned b64 = blocks_for(n64).x;
  hipLaunchKernelGGL(vigp_adam_kernel, dim3(b64 + blocks_for(n32).x), dim3(256), 0, stream, b64, d, s);
  GPL_LAUNCH_CHECK();
  return GPL_OK;
}
