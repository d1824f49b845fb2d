// Gaussian products over sorted points (gauss_tiles.hip): the buffers of a
// product and the pieces shared with the variational step.
#pragma once

#include "common.hpp"
#include "internal.hpp"
#include "tileplan.hpp"

namespace gpl {

// Which side's shapes enter the covariance C_ij (with base I always).
constexpr int kShapesNone = 0, kShapesTarget = 1, kShapesSource = 2, kShapesBoth = 3;

// One side's points along the Hilbert curve (plan_sort): coordinates padded to
// whole 64-point tiles, the caller's indices, and the chunk and subtile boxes.
struct GSorted {
  const float *x, *y;
  const int* perm;
  const float4 *cbox, *sbox;
  int n, nch;
};

struct GTileBufs {
  float* wv;     // [columns][32 nch] source columns with their weights, sorted
  float* form;   // [3][32 nch] forms or shapes of the sources, sorted
  float* reach;  // [nch] largest eigenvalue of a chunk's shapes
  float4 *cdiag, *cdir;  // [nch] its box along the diagonals, reach of its shapes along axes and diagonals
  float4 *sdiag, *sdir;  // the same per 16-target subtile of the targets,
  float* slam;           // and the largest eigenvalue
  float* part;   // [slices][sums][32 nch of the targets] partial sums
};

// -(log2(e)/2) C^{-1} and |C|^{-1/2}.
constexpr float kFormScale = -0.5f * 1.4426950408889634f;
struct Form {
  float xx, xy, yy, rdet;
};
__device__ __forceinline__ Form gauss_form(float cxx, float cxy, float cyy) {
  const float det = fmaf(cxx, cyy, -cxy * cxy), idet = 1.f / det;
  return Form{kFormScale * (cyy * idet), kFormScale * (-cxy * idet), kFormScale * (cxx * idet), rsqrtf(det)};
}

// Sum k (of K) of sorted target i over the slices of part, in slice order.
__device__ __forceinline__ float fold_slices(const float* __restrict__ part, int nslices, int K, int npt, int k,
                                             int i) {
  float s = 0.f;
  for (int q0 = 0; q0 < nslices; q0 += 8) {
    float t[8];  // loads issued together; past the last slice they repeat it and are not added
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = part[((size_t)min(q0 + u, nslices - 1) * K + k) * npt + i];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (q0 + u < nslices) s += t[u];
  }
  return s;
}

GSorted sorted_view(const TilePlan& p);
// Bytes of the buffers of a product of nt targets and ns sources with at most
// `cols` columns held, and their carving.
size_t gauss_tiles_scratch(int nt, int ns, int cols);
int gauss_tiles_carve(int nt, int ns, int cols, void* ws, size_t ws_bytes, GTileBufs& b);
// The product as gauss_product_launch forms it, both sides sorted.
int gauss_tiles_product(const GSorted& T, const float* tz, const float* tw, const GSorted& S, const float* sz,
                        const float* sw, double base, double norm, int nrhs, const float* V, int ldv, float* Y,
                        int ldy, float beta, const GTileBufs& b, hipStream_t stream);
// One column of several layers over shared points, each with its own base covariance.
constexpr int kGaussLayers = 8;
// Per target the partial sums over the sources of G_ij V_j u, into part
// (fold_slices, nslices slices; both set by the call): with the source shapes sz three
// sums, u = 1 and both components of kFormScale C_j^{-1} d, d = target - source, and G_ij
// = |C_j|^{-1/2} exp(-d^T C_j^{-1} d / 2); without (shapes 0) one, u = 1 and
// G_ij = exp(-d^2 / (2 base)).
struct GaussLayerSums {
  GSorted T;
  int shapes;
  double base;
  float* part;
  int nslices;
};
size_t gauss_layers_scratch(const int* nt, int ns, int nl);
int gauss_layers_sums(GaussLayerSums* layers, int nl, const GSorted& S, const float* sz, const float* V, void* scratch,
                      size_t bytes, hipStream_t stream);
// f += sum over the layers of T_k V_k, T_k from sources without shapes in the caller's
// order (S.w given) to the targets T with the shapes tz (caller's order; layers with
// shapes 0: without), and tg, five arrays of T.n floats: the adjoint towards the
// targets per unit of dF/df (two components of the position, three of the shape).
// far_count[k] (device) is zero before the launch.
struct GaussLayer {
  GSide S;
  int shapes;
  double base, norm;
  const float* V;
};
size_t gauss_ordered_scratch(int nt, const int* ns, int nl);
int gauss_ordered_launch(const GSorted& T, const float* tz, const GaussLayer* layers, int nl, float* f, float* tg,
                         int* far_count, void* scratch, size_t bytes, hipStream_t stream);
// The product from the caller's order: sorts the points in the workspace (0 bytes
// where none of these sizes is sorted).
bool gauss_pair_sorted(int nt, int ns, bool tshapes, bool sshapes, bool same, int nrhs);
bool gauss_pair_sorted(const GSide& T, const GSide& S, int nrhs);
size_t gauss_pair_workspace(int nt, int ns, bool same, int nrhs);
int gauss_pair_product(const GSide& T, const GSide& S, double base, double norm, int nrhs, const float* V, int ldv,
                       float* Y, int ldy, float beta, void* ws, size_t ws_bytes, hipStream_t stream,
                       const PlanSide* side = nullptr);

}  // namespace gpl
