// Gaussian products over sorted points with the pairs that are exactly zero left
// out. The sums are those of the dense products of gauss.hip,
//   sum_j ws_j |C_ij|^{-1/2} exp(-d^T C_ij^{-1} d / 2) V_j  (and their moments in C^{-1} d),
// C_ij = Zt_i + Zs_j + base I, for the transmission matrix of Sec. 3.4 (eq.
// "transmission"), the windowed kernel of Sec. 3.2 (eq. "covariance") and the
// variational step built on them.
//
// Both sides are taken along a Hilbert curve of their positions (plan_sort). For any
// direction e, d^T C^{-1} d >= (e.d)^2 / (e^T C e), so a pair of boxes with gap g along
// e has at least g^2 / (base + the largest e^T Z e of both boxes' shapes) for every
// pair in it, and g^2 / lambda for its gap in the plane, lambda the largest eigenvalue.
// v_exp_f32 returns zero below an argument of -126.5, so a 16-target x 32-source pair
// of boxes where (log2(e)/2) times one of these exceeds 127 holds exact zeros only and
// is not evaluated: the sum over the rest is the sum over all pairs up to its order.
// Directions: the axes and the diagonals (traced pixels are long and thin where the
// image is magnified; with the eigenvalue alone, 15% of the pairs of 40,000 traced
// points were evaluated for 12.9 at l = 0.04 and 5.6 for 3.4 at l = 0.01). A chunk
// with a non-finite position, shape, weight or column value, or a shape whose
// covariance is not positive definite, is never left out.
//
// Work: a workgroup of four waves takes 64 targets and every kslices-th chunk of
// 32 sources (strided, since the live chunks of a tile lie together along the
// curve), lists its live chunks with the mask of the four 16-target subtiles that
// see each, and deals them to the waves in turn. A lane holds one target of each
// subtile and 8 of the chunk's sources. Partial sums go to part[slice][sum][target]
// and are added in slice order by a second kernel: a fixed order, so results do
// not vary between runs. Slices keep the tiles whose shapes reach far (next to
// the lens centre one sees every chunk) from being the launch's tail.
//
// Bound by FP32 issue (8 to 19 VALU instructions and one or two transcendentals a
// pair). At 40,000 traced points and l = 0.04 one sum with shapes on one side takes
// 70 us (84 with the eigenvalue's test alone, 636 in the all-pairs kernel); three sums
// of two such layers (l = 0.01 and 0.04) and one of a 40 x 40 grid's 103 us together
// (123). Shapes on both sides, three columns, 16,384 points, l = 0.04: 120 us (178 with
// that test, four columns held and the exponent's factor outside the shapes).
#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "gauss_tiles.hpp"
#include "internal.hpp"
#include "tileplan.hpp"

namespace gpl {

constexpr int kTWaves = 4;                     // waves per workgroup
constexpr int kTBatch = 4;                     // box tests of a lane in a round
constexpr int kTList = kTWaves * kTBatch * 64; // chunks tested per round
constexpr float kZeroArg = 127.f;              // exp2(-kZeroArg) is exactly zero, with margin for rounding

// Pairs below which a product of points in the caller's order is never sorted first
// (shapes on one side or none, on both); above them gauss_pair_sorted weighs the two.
constexpr long long kSortedPairs = 3LL << 25, kSortedPairsBoth = 1LL << 22;
constexpr int kEntryShift = 28;                // list entries: chunk below, subtile mask above
constexpr uint32_t kEntryChunk = (1u << kEntryShift) - 1u;

static_assert(kRowTile == 64 && kSubTile == 16 && kChunk == 32, "the lane layout below");

__device__ __forceinline__ float finite_or_inf(float v) { return v < INFINITY ? v : INFINITY; }  // NaN -> inf

// Upper bound of the largest eigenvalue of the shape (zxx, zxy, zyy); infinite
// when the shape with the covariance base_min added is not positive definite.
__device__ __forceinline__ float shape_reach(float zxx, float zxy, float zyy, float base_min) {
  const float cxx = zxx + base_min, cyy = zyy + base_min;
  if (!(cxx > 0.f && cyy > 0.f && cxx * cyy > zxy * zxy)) return INFINITY;
  const float h = 0.5f * (zxx - zyy);
  return finite_or_inf(fmaxf(0.f, (0.5f * (zxx + zyy) + sqrtf(h * h + zxy * zxy)) * 1.00001f));
}

// The same along the axes and the diagonals: upper bounds of e^T Z e for e = x, y,
// (x + y)/sqrt 2 and (x - y)/sqrt 2, with lam the largest eigenvalue's.
struct Reach {
  float4 dir;
  float lam;
};
__device__ __forceinline__ Reach all_reach(float v) { return Reach{make_float4(v, v, v, v), v}; }
__device__ __forceinline__ Reach shape_reaches(float zxx, float zxy, float zyy, float base_min) {
  const float lam = shape_reach(zxx, zxy, zyy, base_min);
  if (!(lam < INFINITY)) return all_reach(INFINITY);
  const float e = 1e-5f * (fabsf(zxx) + fabsf(zyy) + fabsf(zxy)), h = 0.5f * (zxx + zyy);
  return Reach{make_float4(fmaxf(0.f, zxx) + e, fmaxf(0.f, zyy) + e, fmaxf(0.f, h + zxy) + e, fmaxf(0.f, h - zxy) + e),
               lam};
}
template <int W>  // over each W lanes
__device__ __forceinline__ Reach join_reach(Reach r) {
  for (int off = W / 2; off > 0; off >>= 1) {
    r.dir.x = fmaxf(r.dir.x, __shfl_xor(r.dir.x, off, W));
    r.dir.y = fmaxf(r.dir.y, __shfl_xor(r.dir.y, off, W));
    r.dir.z = fmaxf(r.dir.z, __shfl_xor(r.dir.z, off, W));
    r.dir.w = fmaxf(r.dir.w, __shfl_xor(r.dir.w, off, W));
    r.lam = fmaxf(r.lam, __shfl_xor(r.lam, off, W));
  }
  return r;
}

// Box along the diagonals, (x + y)/sqrt 2 and (x - y)/sqrt 2, of the live points of
// each W lanes, widened by the rounding of these sums; infinite when one is not finite.
template <int W>
__device__ __forceinline__ float4 diagonal_box(float x, float y, bool live) {
  constexpr float kHalfRoot = 0.70710678f, kRound = 4e-7f;
  const float u = (x + y) * kHalfRoot, v = (x - y) * kHalfRoot, eu = kRound * fabsf(u), ev = kRound * fabsf(v);
  float4 q = make_float4(u - eu, u + eu, v - ev, v + ev);
  if (!(isfinite(u) && isfinite(v))) q = make_float4(-INFINITY, INFINITY, -INFINITY, INFINITY);
  if (!live) q = make_float4(INFINITY, -INFINITY, INFINITY, -INFINITY);
  for (int off = W / 2; off > 0; off >>= 1) {
    q.x = fminf(q.x, __shfl_xor(q.x, off, W));
    q.y = fmaxf(q.y, __shfl_xor(q.y, off, W));
    q.z = fminf(q.z, __shfl_xor(q.z, off, W));
    q.w = fmaxf(q.w, __shfl_xor(q.w, off, W));
  }
  return q;
}

// Are all pairs of two boxes exact zeros? a, b: the boxes, da, db: along the
// diagonals; r: base plus the reaches of both (kAxes 0: r.lam alone is looked at). An
// infinite reach (something not finite) is never left out, also where a squared gap
// overflows: so no pair at equality.
template <bool kAxes>
__device__ __forceinline__ bool boxes_zero(const float4& a, const float4& da, const float4& b, const float4& db,
                                           const Reach& r) {
  const float gx = fmaxf(0.f, fmaxf(b.x - a.y, a.x - b.y)), gy = fmaxf(0.f, fmaxf(b.z - a.w, a.z - b.w));
  const float x2 = -kFormScale * (gx * gx), y2 = -kFormScale * (gy * gy);
  bool zero = x2 + y2 > kZeroArg * r.lam;
  if (kAxes) {
    const float gu = fmaxf(0.f, fmaxf(db.x - da.y, da.x - db.y)), gv = fmaxf(0.f, fmaxf(db.z - da.w, da.z - db.w));
    zero = zero || x2 > kZeroArg * r.dir.x || y2 > kZeroArg * r.dir.y ||
           -kFormScale * (gu * gu) > kZeroArg * r.dir.z || -kFormScale * (gv * gv) > kZeroArg * r.dir.w;
  }
  return zero;
}
__device__ __forceinline__ Reach add_reach(float base, const float4& d0, float l0, const float4& d1, float l1) {
  return Reach{make_float4(base + d0.x + d1.x, base + d0.y + d1.y, base + d0.z + d1.z, base + d0.w + d1.w),
               base + l0 + l1};
}

// In the both-sided form shapes and base are held times kBothScale, which makes
// d^T C^{-1} d the exponent; the determinant's root is smaller by it.
constexpr float kBothScale = -1.f / kFormScale;

// Source side in sorted order: columns ws_j V_j (times |C_j|^{-1/2} when the
// shapes are the sources' alone), the forms or shapes, and per chunk its diagonal box
// and the reach of its shapes. Thread j handles sorted source j < npad; the padding
// has zero columns.
template <int MODE>
__device__ __forceinline__ void gauss_prep_source(int j, const GSorted& S, const float* __restrict__ z,
                                                  const float* __restrict__ w, const float* __restrict__ V, int ldv,
                                                  int nc, float base, const GTileBufs& b) {
  const int npad = S.nch * kChunk;
  if (j >= npad) return;  // whole waves: npad is a multiple of 64
  const bool live = j < S.n;
  const int jj = live ? S.perm[j] : 0;
  float scale = live ? (w ? w[jj] : 1.f) : 0.f;
  Reach r = all_reach(0.f);
  if (MODE == kShapesSource || MODE == kShapesBoth) {
    const float zxx = live && z ? z[jj] : 0.f, zxy = live && z ? z[S.n + jj] : 0.f,
                zyy = live && z ? z[2 * (size_t)S.n + jj] : 0.f;
    if (MODE == kShapesSource) {
      const Form f = gauss_form(zxx + base, zxy, zyy + base);
      b.form[j] = f.xx;
      b.form[npad + j] = f.xy;
      b.form[2 * npad + j] = f.yy;
      scale *= f.rdet;
      r = shape_reaches(zxx, zxy, zyy, base);
    } else {
      b.form[j] = kBothScale * zxx;
      b.form[npad + j] = kBothScale * zxy;
      b.form[2 * npad + j] = kBothScale * zyy;
      r = shape_reaches(zxx, zxy, zyy, 0.5f * base);
    }
  }
  for (int c = 0; c < nc; ++c) {
    const float v = live ? scale * V[(size_t)c * ldv + jj] : 0.f;
    b.wv[(size_t)c * npad + j] = v;
    if (!isfinite(v)) r = all_reach(INFINITY);
  }
  r = join_reach<kChunk>(r);
  const float4 q = diagonal_box<kChunk>(S.x[j], S.y[j], live);
  if ((j & (kChunk - 1)) == 0) {
    b.reach[j / kChunk] = r.lam;
    b.cdir[j / kChunk] = r.dir;
    b.cdiag[j / kChunk] = q;
  }
}

// Target side: per 16-target subtile its diagonal box and the reach of its shapes.
template <int MODE>
__device__ __forceinline__ void gauss_prep_target(int i, const GSorted& T, const float* __restrict__ z, float base,
                                                  const GTileBufs& b) {
  if (i >= T.nch * kChunk) return;
  const bool live = i < T.n;
  Reach r = all_reach(0.f);
  if ((MODE == kShapesTarget || MODE == kShapesBoth) && live) {
    const int ii = T.perm[i];
    r = shape_reaches(z[ii], z[T.n + ii], z[2 * (size_t)T.n + ii], MODE == kShapesTarget ? base : 0.5f * base);
  }
  r = join_reach<kSubTile>(r);
  const float4 q = diagonal_box<kSubTile>(T.x[i], T.y[i], live);
  if ((i & (kSubTile - 1)) == 0) {
    b.slam[i / kSubTile] = r.lam;
    b.sdir[i / kSubTile] = r.dir;
    b.sdiag[i / kSubTile] = q;
  }
}

// Both, the second half of the launch (blockIdx.y 1) the targets.
template <int MODE>
__global__ __launch_bounds__(256) void gauss_prep_kernel(GSorted T, const float* __restrict__ tz, GSorted S,
                                                         const float* __restrict__ z, const float* __restrict__ w,
                                                         const float* __restrict__ V, int ldv, int nc, float base,
                                                         GTileBufs b) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (blockIdx.y == 0) gauss_prep_source<MODE>(j, S, z, w, V, ldv, nc, base, b);
  else gauss_prep_target<MODE>(j, T, tz, base, b);
}

// Sums held per target: NC columns, or (MOM) the sum and its first moments in
// the scaled C^{-1} d.
template <bool MOM, int NC>
constexpr int kSums = MOM ? 3 : NC;

template <int MODE, bool MOM, int NC>
__device__ __forceinline__ void gauss_tiles_body(int tile, int slice, int nslices, const GSorted& T,
                                                 const float* __restrict__ tz, const GSorted& S, float base,
                                                 const GTileBufs& b) {
  constexpr bool kAxes = MODE != kShapesNone;
  const float *__restrict__ wv = b.wv, *__restrict__ form = b.form;
  float* __restrict__ part = b.part;
  constexpr int K = kSums<MOM, NC>;
  __shared__ uint32_t list[kTList];
  __shared__ int cnt_s[kTWaves * kTBatch];
  __shared__ float red[kTWaves][K][kRowTile];
  const int tid = threadIdx.x, lane = tid & 63, wvi = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ri = lane & 15, g = lane >> 4;
  const int npt = T.nch * kChunk, nps = S.nch * kChunk;
  // this lane's target of each subtile
  float xi[kSubsPerTile], yi[kSubsPerTile];
  Form F[kSubsPerTile];  // the target's form (shapes of the targets alone) or its shape (both sides)
#pragma unroll
  for (int t = 0; t < kSubsPerTile; ++t) {
    const int i = tile * kRowTile + t * kSubTile + ri;
    xi[t] = T.x[i];
    yi[t] = T.y[i];
    F[t] = Form{0.f, 0.f, 0.f, 1.f};
    if (MODE == kShapesTarget || MODE == kShapesBoth) {
      const int ii = T.perm[min(i, T.n - 1)];
      const float zxx = tz[ii], zxy = tz[T.n + ii], zyy = tz[2 * (size_t)T.n + ii];
      F[t] = MODE == kShapesTarget ? gauss_form(zxx + base, zxy, zyy + base)
                                   : Form{kBothScale * (zxx + base), kBothScale * zxy, kBothScale * (zyy + base), 1.f};
    }
  }
  const float iso = kFormScale / base;
  float acc[kSubsPerTile][K];
#pragma unroll
  for (int t = 0; t < kSubsPerTile; ++t)
#pragma unroll
    for (int k = 0; k < K; ++k) acc[t][k] = 0.f;

  const int mine = cdiv(S.nch - slice, nslices);  // chunks slice, slice + nslices, ...
  for (int k0 = 0; k0 < mine; k0 += kTList) {
    // the live chunks of this round, in order
    uint32_t e[kTBatch];
    unsigned long long bal[kTBatch];
#pragma unroll
    for (int u = 0; u < kTBatch; ++u) {
      const int kw = k0 + (u * kTWaves + wvi) * 64, k = kw + lane;  // the wave's first and the lane's
      uint32_t mask = 0u;
      e[u] = 0u;
      if (kw < mine) {  // few chunks a slice: one batch
        const int c = min(slice + k * nslices, S.nch - 1);
        const float4 q = S.cbox[c], qd = kAxes ? b.cdiag[c] : q, qr = kAxes ? b.cdir[c] : q;
        const float ls = b.reach[c];
#pragma unroll
        for (int t = 0; t < kSubsPerTile; ++t) {
          const int st = tile * kSubsPerTile + t;  // uniform: the subtile's records come by scalar loads
          const float4 sb = T.sbox[st], sd = kAxes ? b.sdiag[st] : sb, sr = kAxes ? b.sdir[st] : sb;
          const bool zero = boxes_zero<kAxes>(sb, sd, q, qd, add_reach(base, sr, b.slam[st], qr, ls));
          mask |= (zero ? 0u : 1u) << t;
        }
        if (k >= mine) mask = 0u;
        e[u] = (uint32_t)c | (mask << kEntryShift);
      }
      bal[u] = __ballot(mask != 0u);
      if (lane == 0) cnt_s[u * kTWaves + wvi] = __popcll(bal[u]);
    }
    __syncthreads();
    int total = 0, before[kTBatch];
#pragma unroll
    for (int u = 0; u < kTBatch; ++u)
#pragma unroll
      for (int w = 0; w < kTWaves; ++w) {
        if (w == wvi) before[u] = total;
        total += cnt_s[u * kTWaves + w];
      }
#pragma unroll
    for (int u = 0; u < kTBatch; ++u)
      if (e[u] >> kEntryShift) list[before[u] + __popcll(bal[u] & ((1ull << lane) - 1ull))] = e[u];
    __syncthreads();
    for (int p = wvi; p < total; p += kTWaves) {
      const uint32_t ent = (uint32_t)__builtin_amdgcn_readfirstlane((int)list[p]);
      const int j0 = (int)(ent & kEntryChunk) * kChunk + g * 8;
      float xj[8], yj[8], wj[NC][8], fxx[8], fxy[8], fyy[8];
      auto load8 = [](float(&d)[8], const float* s) {
        const float4 a = *reinterpret_cast<const float4*>(s), b = *reinterpret_cast<const float4*>(s + 4);
        d[0] = a.x, d[1] = a.y, d[2] = a.z, d[3] = a.w, d[4] = b.x, d[5] = b.y, d[6] = b.z, d[7] = b.w;
      };
      load8(xj, S.x + j0);
      load8(yj, S.y + j0);
#pragma unroll
      for (int c = 0; c < NC; ++c) load8(wj[c], wv + (size_t)c * nps + j0);
      if (MODE == kShapesSource || MODE == kShapesBoth) {
        load8(fxx, form + j0);
        load8(fxy, form + nps + j0);
        load8(fyy, form + 2 * nps + j0);
      }
#pragma unroll
      for (int t = 0; t < kSubsPerTile; ++t) {
        if (!((ent >> (kEntryShift + t)) & 1u)) continue;
#pragma unroll
        for (int v = 0; v < 8; ++v) {
          const float dx = xi[t] - xj[v], dy = yi[t] - yj[v];
          float val, ux = 0.f, uy = 0.f;
          if (MODE == kShapesNone) {
            val = exp2_fast(iso * fmaf(dx, dx, dy * dy));
          } else if (MODE == kShapesBoth) {
            const float cxx = F[t].xx + fxx[v], cxy = F[t].xy + fxy[v], cyy = F[t].yy + fyy[v];
            const float rd = rsqrtf(fmaf(cxx, cyy, -cxy * cxy));
            const float vx = fmaf(-cxy, dy, cyy * dx), vy = fmaf(-cxy, dx, cxx * dy);
            val = rd * exp2_fast(-(fmaf(dx, vx, dy * vy) * (rd * rd)));
          } else {
            const float a = MODE == kShapesTarget ? F[t].xx : fxx[v], b = MODE == kShapesTarget ? F[t].xy : fxy[v],
                        d = MODE == kShapesTarget ? F[t].yy : fyy[v];
            ux = fmaf(a, dx, b * dy);
            uy = fmaf(b, dx, d * dy);
            val = exp2_fast(fmaf(dx, ux, dy * uy));
          }
          if (MOM) {
            const float gv = val * wj[0][v];
            acc[t][0] += gv;
            acc[t][1 % K] = fmaf(gv, ux, acc[t][1 % K]);
            acc[t][2 % K] = fmaf(gv, uy, acc[t][2 % K]);
          } else {
#pragma unroll
            for (int c = 0; c < NC; ++c) acc[t][c] = fmaf(val, wj[c][v], acc[t][c]);
          }
        }
      }
    }
    __syncthreads();  // the list is rebuilt by the next round
  }
  // the four lanes of a target, then the four waves, in a fixed order
#pragma unroll
  for (int t = 0; t < kSubsPerTile; ++t)
#pragma unroll
    for (int k = 0; k < K; ++k) {
      float v = acc[t][k];
      v += __shfl_xor(v, 16, 64);
      v += __shfl_xor(v, 32, 64);
      if (g == 0) red[wvi][k][t * kSubTile + ri] = v;
    }
  __syncthreads();
  for (int o = tid; o < K * kRowTile; o += 64 * kTWaves) {
    const int k = o / kRowTile, r = o % kRowTile;
    float v = red[0][k][r];
#pragma unroll
    for (int w = 1; w < kTWaves; ++w) v += red[w][k][r];
    part[((size_t)slice * K + k) * npt + tile * kRowTile + r] = v;
  }
}

template <int MODE, bool MOM, int NC>
__global__ __launch_bounds__(64 * kTWaves) void gauss_tiles_kernel(GSorted T, const float* __restrict__ tz, GSorted S,
                                                                   float base, GTileBufs b) {
  gauss_tiles_body<MODE, MOM, NC>(blockIdx.x, blockIdx.y, gridDim.y, T, tz, S, base, b);
}

// Y[c][i] = norm wt_i |C_i|^{-1/2} sum + beta Y[c][i] (the determinant when the
// shapes are the targets' alone).
template <int MODE>
__global__ __launch_bounds__(256) void gauss_finish_kernel(GSorted T, const float* __restrict__ tz,
                                                           const float* __restrict__ tw, float base, float norm,
                                                           const float* __restrict__ part, int nslices, int K,
                                                           float* Y, int ldy, float beta) {
  const int i = blockIdx.x * 256 + threadIdx.x, c = blockIdx.y;
  if (i >= T.n) return;
  const int ii = T.perm[i];
  float f = norm * (tw ? tw[ii] : 1.f);
  if (MODE == kShapesTarget)
    f *= gauss_form(tz[ii] + base, tz[T.n + ii], tz[2 * (size_t)T.n + ii] + base).rdet;
  if (MODE == kShapesNone) f *= rsqrtf(base * base);
  if (MODE == kShapesBoth) f *= kBothScale;
  const float s = f * fold_slices(part, nslices, K, T.nch * kChunk, c, i);
  float* y = Y + (size_t)c * ldy + ii;
  *y = beta != 0.f ? s + beta * *y : s;
}

// About 4096 workgroups, at most 32 slices (each adds its partial sums to the second kernel).
static int tile_slices(const GSorted& T, const GSorted& S) {
  return std::max(1, std::min({32, 4096 / cdiv(T.n, kRowTile), S.nch}));
}

// Columns a kernel holds for nc columns: nc up to four, and eight for five to seven (16,384
// points, shapes of the targets: three columns take 76 us, five 106, eight 107).
static int held_columns(int nc) { return nc > 4 ? 8 : nc; }

template <class C>
static void carve_tiles(C& cv, const GSorted& T, const GSorted& S, int cols, GTileBufs& b) {
  const size_t nps = (size_t)S.nch * kChunk, npt = (size_t)T.nch * kChunk;
  const int held = held_columns(cols);
  b.wv = cv.template take<float>(held * nps);
  b.form = cv.template take<float>(3 * nps);
  b.reach = cv.template take<float>(S.nch);
  b.cdiag = cv.template take<float4>(S.nch);
  b.cdir = cv.template take<float4>(S.nch);
  const size_t subs = (size_t)T.nch * kChunk / kSubTile;
  b.sdiag = cv.template take<float4>(subs);
  b.sdir = cv.template take<float4>(subs);
  b.slam = cv.template take<float>(subs);
  b.part = cv.template take<float>((size_t)tile_slices(T, S) * std::max(held, 3) * npt);
}

static GSorted sorted_sizes(int n) {
  GSorted s{};
  s.n = n;
  s.nch = cdiv(n, kRowTile) * kChunksPerTile;
  return s;
}

GSorted sorted_view(const TilePlan& p) { return GSorted{p.xs, p.ys, p.perm, p.cbox, p.sbox, p.n, p.nch}; }

size_t gauss_tiles_scratch(int nt, int ns, int cols) {
  Sizer s;
  GTileBufs b;
  carve_tiles(s, sorted_sizes(nt), sorted_sizes(ns), cols, b);
  return s.used;
}

int gauss_tiles_carve(int nt, int ns, int cols, void* ws, size_t ws_bytes, GTileBufs& b) {
  GPL_TRY(check_ws(ws, ws_bytes, gauss_tiles_scratch(nt, ns, cols)));
  Carver cv(ws, ws_bytes);
  carve_tiles(cv, sorted_sizes(nt), sorted_sizes(ns), cols, b);
  return cv.ok() ? GPL_OK : check_ws(nullptr, 0, 1);
}

template <int MODE, bool MOM, int NC>
static int tiles_launch(const GSorted& T, const float* tz, const GSorted& S, float base, const GTileBufs& b,
                        int nslices, hipStream_t stream) {
  hipLaunchKernelGGL((gauss_tiles_kernel<MODE, MOM, NC>), dim3(cdiv(T.n, kRowTile), nslices), dim3(64 * kTWaves), 0,
                     stream, T, tz, S, base, b);
  GPL_LAUNCH_CHECK();
  return GPL_OK;
}

template <int MODE>
static int product_cols(const GSorted& T, const float* tz, const float* tw, const GSorted& S, const float* sz,
                        const float* sw, float base, float norm, int nrhs, const float* V, int ldv, float* Y, int ldy,
                        float beta, const GTileBufs& b, hipStream_t stream) {
  const int ns = tile_slices(T, S);
  for (int c0 = 0; c0 < nrhs;) {
    const int nc = std::min(8, nrhs - c0);
    const int held = held_columns(nc);  // those past nc hold anything and are not stored
    hipLaunchKernelGGL(gauss_prep_kernel<MODE>, dim3(cdiv(std::max(S.nch, T.nch) * kChunk, 256), 2), dim3(256), 0,
                       stream, T, tz, S, sz, sw, V + (size_t)c0 * ldv, ldv, nc, base, b);
    GPL_LAUNCH_CHECK();
    switch (held) {
      case 1: GPL_TRY((tiles_launch<MODE, false, 1>(T, tz, S, base, b, ns, stream))); break;
      case 2: GPL_TRY((tiles_launch<MODE, false, 2>(T, tz, S, base, b, ns, stream))); break;
      case 3: GPL_TRY((tiles_launch<MODE, false, 3>(T, tz, S, base, b, ns, stream))); break;
      case 4: GPL_TRY((tiles_launch<MODE, false, 4>(T, tz, S, base, b, ns, stream))); break;
      default: GPL_TRY((tiles_launch<MODE, false, 8>(T, tz, S, base, b, ns, stream))); break;
    }
    hipLaunchKernelGGL(gauss_finish_kernel<MODE>, dim3(cdiv(T.n, 256), nc), dim3(256), 0, stream, T, tz, tw, base,
                       norm, b.part, ns, held, Y + (size_t)c0 * ldy, ldy, beta);
    GPL_LAUNCH_CHECK();
    c0 += nc;
  }
  return GPL_OK;
}

int gauss_tiles_product(const GSorted& T, const float* tz, const float* tw, const GSorted& S, const float* sz,
                        const float* sw, double base, double norm, int nrhs, const float* V, int ldv, float* Y,
                        int ldy, float beta, const GTileBufs& b, hipStream_t stream) {
  const float fb = (float)base, fn = (float)norm;
  if (tz && sz)
    return product_cols<kShapesBoth>(T, tz, tw, S, sz, sw, fb, fn, nrhs, V, ldv, Y, ldy, beta, b, stream);
  if (tz) return product_cols<kShapesTarget>(T, tz, tw, S, sz, sw, fb, fn, nrhs, V, ldv, Y, ldy, beta, b, stream);
  if (sz) return product_cols<kShapesSource>(T, tz, tw, S, sz, sw, fb, fn, nrhs, V, ldv, Y, ldy, beta, b, stream);
  return product_cols<kShapesNone>(T, tz, tw, S, sz, sw, fb, fn, nrhs, V, ldv, Y, ldy, beta, b, stream);
}

// ---- one column of several layers at once
//
// The layers of a source model share the points; each has its own base covariance
// and its own targets (the traced points or the grid). Their launches are one: at a
// thousand points each costs its launch and no more, and at 40,000 the tail of one
// layer's launch is filled by the next layer's work (longest reach first).
struct SumsArgs {
  GSorted S;
  const float *V, *sz;
  struct {
    GSorted T;
    int tiles, slices, shapes;
    float base;
    GTileBufs b;
  } l[kGaussLayers];
};

// blockIdx.y: layer, then the sources (0) or the targets.
__global__ __launch_bounds__(256) void gauss_layers_prep_kernel(SumsArgs A) {
  const auto& L = A.l[blockIdx.y >> 1];
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (blockIdx.y & 1) {
    gauss_prep_target<kShapesNone>(j, L.T, nullptr, L.base, L.b);
  } else if (L.shapes) {
    gauss_prep_source<kShapesSource>(j, A.S, A.sz, nullptr, A.V, 0, 1, L.base, L.b);
  } else {
    gauss_prep_source<kShapesNone>(j, A.S, nullptr, nullptr, A.V, 0, 1, L.base, L.b);
  }
}

__global__ __launch_bounds__(64 * kTWaves) void gauss_layers_kernel(SumsArgs A) {
  const auto& L = A.l[blockIdx.y];
  const int slice = blockIdx.x / L.tiles, tile = blockIdx.x - slice * L.tiles;
  if (slice >= L.slices) return;
  if (L.shapes) gauss_tiles_body<kShapesSource, true, 1>(tile, slice, L.slices, L.T, nullptr, A.S, L.base, L.b);
  else gauss_tiles_body<kShapesNone, false, 1>(tile, slice, L.slices, L.T, nullptr, A.S, L.base, L.b);
}

template <class C>
static void carve_sums(C& cv, const int* nt, int ns, int nl, GTileBufs* b) {
  for (int k = 0; k < nl; ++k) carve_tiles(cv, sorted_sizes(nt[k]), sorted_sizes(ns), 1, b[k]);
}

size_t gauss_layers_scratch(const int* nt, int ns, int nl) {
  Sizer s;
  GTileBufs b[kGaussLayers];
  carve_sums(s, nt, ns, nl, b);
  return s.used;
}

int gauss_layers_sums(GaussLayerSums* layers, int nl, const GSorted& S, const float* sz, const float* V, void* scratch,
                      size_t bytes, hipStream_t stream) {
  GPL_REQUIRE(nl >= 1 && nl <= kGaussLayers, "nl=%d", nl);
  int nt[kGaussLayers], turn[kGaussLayers];
  GTileBufs b[kGaussLayers];
  for (int k = 0; k < nl; ++k) {
    nt[k] = layers[k].T.n;
    turn[k] = k;
  }
  Carver cv(scratch, bytes);
  carve_sums(cv, nt, S.n, nl, b);
  if (!cv.ok()) return check_ws(nullptr, 0, 1);
  std::stable_sort(turn, turn + nl, [&](int x, int y) { return layers[x].base > layers[y].base; });
  SumsArgs A{};
  A.S = S;
  A.V = V;
  A.sz = sz;
  int blocks = 0, npad = S.nch * kChunk;
  for (int q = 0; q < nl; ++q) {
    GaussLayerSums& L = layers[turn[q]];
    L.part = b[turn[q]].part;
    L.nslices = tile_slices(L.T, S);
    A.l[q] = {L.T, cdiv(L.T.n, kRowTile), L.nslices, L.shapes, (float)L.base, b[turn[q]]};
    blocks = std::max(blocks, A.l[q].tiles * L.nslices);
    npad = std::max(npad, L.T.nch * kChunk);
  }
  hipLaunchKernelGGL(gauss_layers_prep_kernel, dim3(cdiv(npad, 256), 2 * nl), dim3(256), 0, stream, A);
  GPL_LAUNCH_CHECK();
  hipLaunchKernelGGL(gauss_layers_kernel, dim3(blocks, nl), dim3(64 * kTWaves), 0, stream, A);
  GPL_LAUNCH_CHECK();
  return GPL_OK;
}

// ---- one column, sources in the caller's order
//
// The transmission T y of the variational step with the sums its adjoint towards
// the targets needs. The targets are sorted, the sources stay in the caller's
// order, and the sum over them has a fixed one: eight shares of whole 64-point steps,
// each added up source by source, then the shares in order. Chunks of eight
// consecutive sources whose terms are exact zeros are left out, which changes no bit.
// (The log-likelihood is a sum of squares of small differences of these fluxes in
// FP64: another order of the sum moves it by some 1e-9, within its own error but
// visible from one version to the next.)
//
// A wave takes 16 targets and one share: lane 4 t + q forms the terms of target t
// and source q of every four, and the sum goes round the four lanes of a target,
// each adding its own term (DPP moves within the quad).
// Several images of one source region fall into one share (a band of image rows),
// so the longest waves see all of their share: with 64 targets a wave these took
// 430 us at l = 0.04 of a launch whose work is worth 150. For the same reason each
// wave is a workgroup of its own, and a second kernel adds the shares: waves that
// wait for the longest share of their targets keep others from being started.
// Bound by issue, about 27 VALU instructions and one exp for 64 pairs: 204 us for two
// layers of 40,000 points (l = 0.01 and 0.04) and one of a 40 x 40 grid together, 231 us
// with the eigenvalue's test alone; the all-pairs product took 580 us a layer and its
// adjoint towards the targets, formed here with it, another 767 us.
//
// Targets whose shapes reach far (next to the lens centre) would have their
// neighbours evaluate every source too. Those with a shape beyond kFarReach base
// are listed and taken by workgroups of their own, the sources dealt to the
// threads and the sums folded in a tree (fewer than one target in a hundred, so
// the order of their sums does not matter to the likelihood).

constexpr int kOChunk = 8;     // consecutive sources of a box
constexpr int kOTargets = 16;  // targets of a wave, four lanes each
constexpr int kOWaves = 8;    // shares of the sources, one wave each
constexpr float kFarReach = 8.f;
constexpr int kFarBlocks = 2048;  // waves that take the listed targets in turn
static_assert(64 % kOChunk == 0 && kOChunk % 4 == 0 && kOTargets == kSubTile, "whole chunks and quads");

static __host__ __device__ int ordered_share(int n) { return cdiv(cdiv(n, 64), kOWaves) * (64 / kOChunk); }

struct OrderedBufs {
  float4 *src, *box, *cdiag;  // sources, and the boxes of their chunks
  float4 *sdiag, *sdir;       // per 16 targets: diagonal box and reach of their shapes
  float* slam;
  int* far;                   // the listed targets
  unsigned* sfar;             // per 16 targets: which of them are listed (the one decision on it)
  float* part;
};
struct OrderedArgs {
  GSorted T;
  const float* tz;
  int tiles, nl;
  int turn[kGaussLayers];  // launch order of the layers
  struct {
    const float *x, *y, *w, *V;
    int ns, shapes;
    float base, norm;
    int* far_count;
    OrderedBufs b;
  } l[kGaussLayers];
};

// Layer blockIdx.y. Source j: (x, y, weight, column value), zeros past n, and the
// box of its chunk, infinite when one of them is not finite in it. Sorted target j:
// listed in far when its shape reaches far (the order of the list does not enter
// any result).
__global__ __launch_bounds__(256) void ordered_prep_kernel(OrderedArgs A) {
  const auto& L = A.l[blockIdx.y];
  const int n = L.ns;
  const float *__restrict__ x = L.x, *__restrict__ y = L.y, *__restrict__ w = L.w, *__restrict__ V = L.V;
  const float* __restrict__ tz = A.tz;
  const int j = blockIdx.x * 256 + threadIdx.x, npad = round_up(n, kOChunk);
  if (L.shapes && j < A.T.nch * kChunk) {
    Reach r = all_reach(0.f);
    bool live = j < A.T.n, listed = false;
    if (live) {
      const int jj = A.T.perm[j];
      r = shape_reaches(tz[jj], tz[A.T.n + jj], tz[2 * (size_t)A.T.n + jj], L.base);
      listed = r.lam > kFarReach * L.base;
      if (listed) {
        L.b.far[atomicAdd(L.far_count, 1)] = j;
        r = all_reach(0.f);
        live = false;
      }
    }
    const unsigned long long bal = __ballot(listed);
    r = join_reach<kSubTile>(r);
    const float4 q = diagonal_box<kSubTile>(A.T.x[j], A.T.y[j], live);
    if ((j & (kSubTile - 1)) == 0) {
      L.b.sfar[j / kSubTile] = (unsigned)(bal >> (j & 63)) & ((1u << kSubTile) - 1u);
      L.b.slam[j / kSubTile] = r.lam;
      L.b.sdir[j / kSubTile] = r.dir;
      L.b.sdiag[j / kSubTile] = q;
    }
  }
  float4 q = make_float4(INFINITY, -INFINITY, INFINITY, -INFINITY), s = make_float4(0.f, 0.f, 0.f, 0.f);
  bool ok = false;
  if (j < n) {
    s = make_float4(x[j], y[j], w[j], V[j]);
    ok = isfinite(s.x) && isfinite(s.y) && isfinite(s.z) && isfinite(s.w);
    q = ok ? make_float4(s.x, s.x, s.y, s.y) : make_float4(-INFINITY, INFINITY, -INFINITY, INFINITY);
  }
  if (j < npad) L.b.src[j] = s;
  for (int off = kOChunk / 2; off > 0; off >>= 1) {
    q.x = fminf(q.x, __shfl_xor(q.x, off, kOChunk));
    q.y = fmaxf(q.y, __shfl_xor(q.y, off, kOChunk));
    q.z = fminf(q.z, __shfl_xor(q.z, off, kOChunk));
    q.w = fmaxf(q.w, __shfl_xor(q.w, off, kOChunk));
  }
  const float4 d = diagonal_box<kOChunk>(ok ? s.x : INFINITY, s.y, j < n);
  if (j < npad && (j & (kOChunk - 1)) == 0) {
    L.b.box[j / kOChunk] = q;
    L.b.cdiag[j / kOChunk] = d;
  }
}

// One target of the ordered product: its form, and the terms of one source.
template <bool kShapes>
struct OrderedTarget {
  static constexpr int K = kShapes ? 6 : 3;
  float x, y, ixx, ixy, iyy, rdet;
  float acc[K];
  __device__ __forceinline__ void init(float xi, float yi, float txx, float txy, float tyy, float base) {
    x = xi;
    y = yi;
    const float cxx = txx + base, cxy = txy, cyy = tyy + base;
    const float det = fmaf(cxx, cyy, -cxy * cxy), idet = 1.f / det;
    ixx = cyy * idet;
    ixy = -cxy * idet;
    iyy = cxx * idet;
    rdet = rsqrtf(det);
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] = 0.f;
  }
  // the weighted Gaussian of source s, its moments added
  __device__ __forceinline__ float term(const float4& s) {
    const float dx = x - s.x, dy = y - s.y;
    const float ux = kShapes ? fmaf(ixx, dx, ixy * dy) : ixx * dx;
    const float uy = kShapes ? fmaf(ixy, dx, iyy * dy) : iyy * dy;
    const float val = s.z * exp2_fast(kFormScale * fmaf(dx, ux, dy * uy));
    const float gv = val * s.w;
    const float gx = gv * ux, gy = gv * uy;
    acc[1] += gx;
    acc[2] += gy;
    if (kShapes) {
      acc[3 % K] = fmaf(gx, ux, acc[3 % K]);
      acc[4 % K] = fmaf(gx, uy, acc[4 % K]);
      acc[5 % K] = fmaf(gy, uy, acc[5 % K]);
    }
    return val;
  }
  // f += norm |C|^{-1/2} sum, and tg: -sum G C^{-1} d for the positions and, with
  // shapes, sum G (C^{-1} d d^T C^{-1} - C^{-1}) / 2 (xx, xy, yy) with the same factor.
  __device__ __forceinline__ void add(float norm, float& f, float (&tg)[5]) const {
    const float c = norm * rdet, h = 0.5f * c;
    f = fmaf(c, acc[0], f);
    tg[0] -= c * acc[1];
    tg[1] -= c * acc[2];
    if (kShapes) {
      tg[2] += h * (acc[3 % K] - ixx * acc[0]);
      tg[3] += h * (acc[4 % K] - ixy * acc[0]);
      tg[4] += h * (acc[5 % K] - iyy * acc[0]);
    }
  }
};

// Each four lanes: the value of the lane before (lane 0 takes lane 3's).
__device__ __forceinline__ float quad_next(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x93, 0xf, 0xf, true));
}

// Workgroup (wave) b < 8 tiles: share b / tiles of the sources for the 16 sorted
// targets of tile b % tiles (a share's waves go round the XCDs: the shares that
// hold the images are several times the work of the others). The rest (with
// shapes): wave q takes eighth q % 8 of the sources of listed target q / 8.
template <bool kShapes>
__device__ __forceinline__ void gauss_ordered_body(const GSorted& T, int tiles, const float* __restrict__ tz, int ns,
                                                   const OrderedBufs& b, float base,
                                                   const int* __restrict__ far_count) {
  const float4* __restrict__ src = b.src;
  const int* __restrict__ far = b.far;
  float* __restrict__ part = b.part;
  using Target = OrderedTarget<kShapes>;
  constexpr int K = Target::K;
  const int lane = threadIdx.x, wv = blockIdx.x / tiles, tile = blockIdx.x % tiles, npt = T.nch * kChunk;
  const int quad = lane & 3;
  Target t;
  if (kShapes && wv >= kOWaves) {
    const int cnt = *far_count * kOWaves, first = tiles * kOWaves;
    for (int q = blockIdx.x - first; q < cnt; q += kFarBlocks) {
      const int i = far[q / kOWaves], ii = T.perm[i], w = q % kOWaves;
      t.init(T.x[i], T.y[i], tz[ii], tz[T.n + ii], tz[2 * (size_t)T.n + ii], base);
      for (int j = w * 64 + lane; j < ns; j += 64 * kOWaves) {
        const float4 s = src[j];
        t.acc[0] = fmaf(t.term(s), s.w, t.acc[0]);
      }
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const float v = warp_sum(t.acc[k]);
        if (lane == 0) part[((size_t)w * K + k) * npt + i] = v;
      }
    }
    return;
  }
  const int i = tile * kOTargets + (lane >> 2);
  bool live = i < T.n;
  const int ii = T.perm[min(i, T.n - 1)];
  float txx = 0.f, txy = 0.f, tyy = 0.f;
  Reach r = all_reach(base);
  const float4 rb = T.sbox[tile];
  float4 rd = rb;
  if (kShapes) {
    txx = tz[ii];
    txy = tz[T.n + ii];
    tyy = tz[2 * (size_t)T.n + ii];
    if ((b.sfar[tile] >> (lane >> 2)) & 1u) live = false;  // listed
    rd = b.sdiag[tile];
    r = add_reach(base, b.sdir[tile], b.slam[tile], make_float4(0.f, 0.f, 0.f, 0.f), 0.f);
  }
  t.init(T.x[i], T.y[i], txx, txy, tyy, base);
  const int nch = cdiv(ns, kOChunk), share = ordered_share(ns);
  const int cend = min(nch, (wv + 1) * share);
  for (int c0 = wv * share; c0 < cend; c0 += 64) {
    const int c = min(c0 + lane, nch - 1);
    const float4 q = b.box[c], qd = kShapes ? b.cdiag[c] : q;
    const bool zero = boxes_zero<kShapes>(rb, rd, q, qd, r);
    unsigned long long m = __ballot(c0 + lane < cend && !zero);
    while (m != 0ull) {
      const int j0 = (c0 + __ffsll((long long)m) - 1) * kOChunk;
      m &= m - 1ull;
      float4 s[kOChunk / 4];
#pragma unroll
      for (int v = 0; v < kOChunk / 4; ++v) s[v] = src[j0 + 4 * v + quad];
#pragma unroll
      for (int v = 0; v < kOChunk / 4; ++v) {
        // the sum so far is lane 0's: it takes its term, lane 1 the next, ...
        const float val = t.term(s[v]);
#pragma unroll
        for (int k = 0; k < 4; ++k) t.acc[0] = quad_next(fmaf(val, s[v].w, t.acc[0]));
      }
    }
  }
#pragma unroll
  for (int k = 1; k < K; ++k) {  // the moments of the four lanes (the sum itself is in lane 0)
    t.acc[k] += __shfl_xor(t.acc[k], 1, 64);
    t.acc[k] += __shfl_xor(t.acc[k], 2, 64);
  }
  if (quad != 0 || !live) return;
#pragma unroll
  for (int k = 0; k < K; ++k) part[((size_t)wv * K + k) * npt + i] = t.acc[k];
}

__global__ __launch_bounds__(64) void gauss_ordered_kernel(OrderedArgs A) {
  const auto& L = A.l[A.turn[blockIdx.y]];
  if (L.shapes) {
    gauss_ordered_body<true>(A.T, A.tiles, A.tz, L.ns, L.b, L.base, L.far_count);
  } else if ((int)blockIdx.x < A.tiles * kOWaves) {
    gauss_ordered_body<false>(A.T, A.tiles, nullptr, L.ns, L.b, L.base, nullptr);
  }
}

// One layer of the end: the shares added in order.
template <bool kShapes>
__device__ __forceinline__ void ordered_finish(const GSorted& T, int i, int ii, const float* __restrict__ tz,
                                               float base, float norm, const float* __restrict__ part, float& f,
                                               float (&tg)[5]) {
  using Target = OrderedTarget<kShapes>;
  constexpr int K = Target::K;
  const int npt = T.nch * kChunk;
  Target t;
  t.init(T.x[i], T.y[i], kShapes ? tz[ii] : 0.f, kShapes ? tz[T.n + ii] : 0.f, kShapes ? tz[2 * (size_t)T.n + ii] : 0.f,
         base);
  float v[kOWaves][K];
#pragma unroll
  for (int w = 0; w < kOWaves; ++w)
#pragma unroll
    for (int k = 0; k < K; ++k) v[w][k] = part[((size_t)w * K + k) * npt + i];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    t.acc[k] = v[0][k];
#pragma unroll
    for (int w = 1; w < kOWaves; ++w) t.acc[k] += v[w][k];
  }
  t.add(norm, f, tg);
}

// f += the layers in their order, tg = their adjoint towards the targets.
__global__ __launch_bounds__(256) void ordered_finish_kernel(OrderedArgs A, float* f, float* tg) {
  const int i = blockIdx.x * 256 + threadIdx.x, n = A.T.n;
  if (i >= n) return;
  const int ii = A.T.perm[i];
  float fi = f[ii], t[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
  for (int k = 0; k < A.nl; ++k) {
    const auto& L = A.l[k];
    if (L.shapes) ordered_finish<true>(A.T, i, ii, A.tz, L.base, L.norm, L.b.part, fi, t);
    else ordered_finish<false>(A.T, i, ii, nullptr, L.base, L.norm, L.b.part, fi, t);
  }
  f[ii] = fi;
#pragma unroll
  for (int k = 0; k < 5; ++k) tg[(size_t)k * n + ii] = t[k];
}

template <class C>
static void carve_ordered(C& cv, int nt, const int* ns, int nl, OrderedBufs* b) {
  for (int k = 0; k < nl; ++k) {
    b[k].src = cv.template take<float4>(round_up(ns[k], kOChunk));
    b[k].box = cv.template take<float4>(cdiv(ns[k], kOChunk));
    b[k].cdiag = cv.template take<float4>(cdiv(ns[k], kOChunk));
    const size_t subs = (size_t)round_up(nt, kRowTile) / kSubTile;
    b[k].sdiag = cv.template take<float4>(subs);
    b[k].sdir = cv.template take<float4>(subs);
    b[k].slam = cv.template take<float>(subs);
    b[k].far = cv.template take<int>(nt);
    b[k].sfar = cv.template take<unsigned>(subs);
    b[k].part = cv.template take<float>((size_t)kOWaves * 6 * round_up(nt, kRowTile));
  }
}

size_t gauss_ordered_scratch(int nt, const int* ns, int nl) {
  Sizer s;
  OrderedBufs b[kGaussLayers];
  carve_ordered(s, nt, ns, nl, b);
  return s.used;
}

int gauss_ordered_launch(const GSorted& T, const float* tz, const GaussLayer* layers, int nl, float* f, float* tg,
                         int* far_count, void* scratch, size_t bytes, hipStream_t stream) {
  GPL_REQUIRE(nl >= 1 && nl <= kGaussLayers, "nl=%d", nl);
  OrderedArgs A{};
  A.T = T;
  A.tz = tz;
  A.tiles = cdiv(T.n, kOTargets);
  A.nl = nl;
  int ns[kGaussLayers], prep = 1;
  OrderedBufs b[kGaussLayers];
  bool shapes = false;
  for (int k = 0; k < nl; ++k) {
    ns[k] = layers[k].S.n;
    A.turn[k] = k;
    prep = std::max({prep, round_up(ns[k], kOChunk), layers[k].shapes ? round_up(T.n, kRowTile) : 0});
    shapes = shapes || layers[k].shapes;
  }
  Carver cv(scratch, bytes);
  carve_ordered(cv, T.n, ns, nl, b);
  if (!cv.ok()) return check_ws(nullptr, 0, 1);
  for (int k = 0; k < nl; ++k) {
    const GaussLayer& q = layers[k];
    A.l[k] = {q.S.x, q.S.y, q.S.w, q.V, q.S.n, q.shapes, (float)q.base, (float)q.norm, far_count + k, b[k]};
  }
  std::stable_sort(A.turn, A.turn + nl, [&](int p, int q) { return layers[p].base > layers[q].base; });
  hipLaunchKernelGGL(ordered_prep_kernel, dim3(cdiv(prep, 256), nl), dim3(256), 0, stream, A);
  GPL_LAUNCH_CHECK();
  hipLaunchKernelGGL(gauss_ordered_kernel, dim3(A.tiles * kOWaves + (shapes ? kFarBlocks : 0), nl), dim3(64), 0, stream,
                     A);
  GPL_LAUNCH_CHECK();
  hipLaunchKernelGGL(ordered_finish_kernel, dim3(cdiv(T.n, 256)), dim3(256), 0, stream, A, f, tg);
  GPL_LAUNCH_CHECK();
  return GPL_OK;
}

template <class C>
static void carve_pair(C& cv, int nt, int ns, bool same, int cols, TilePlan& pt, TilePlan& ps, char*& rest,
                       size_t& bytes) {
  sort_carve(cv, nt, pt);
  if (!same) sort_carve(cv, ns, ps);
  bytes = gauss_tiles_scratch(nt, ns, cols);
  rest = cv.template take<char>(bytes);
}

// Whether a product is sorted first: whether the sorts of its points cost less than all
// pairs do. In us, fitted to sizes of 64 to 400,000 points on either side at l = 0.04
// over a field of 5: all pairs go by 1,024 sources (by steps of 512 in a single round of
// workgroups) for each 16,384 targets, and a set's sort costs by its points up to some
// 5,600 and is bound by launches beyond. The long side counts as much as the number of
// pairs. One column with shapes of the targets takes, all pairs and sorted, 57 and 64 us
// for 10,000 points (one set), 90 and 70 for 16,384; for 40,000 targets 17 and 72 with
// 1,024 sources, 59 and 87 with 4,096, 142 and 109 with 10,000; 116 and 183 for 400,000
// and 1,024. With shapes on both sides and three columns: 56 and 40 for 2,500 (one set), 24
// and 61 for 4,096 targets and 1,024 sources, 82 and 55 for 1,024 and 4,096; with eight 134
// and 145 for 40,000 and 2,500. Where the
// lengthscale is not small against the field fewer terms are zero: at l = 1 the sorted
// product takes up to 1.4 times as long as all pairs near the line.
static double sort_us(int n) { return std::min(5.0 + n / 160.0, 40.0) + 3.5e-4 * n; }

bool gauss_pair_sorted(int nt, int ns, bool tshapes, bool sshapes, bool same, int nrhs) {
  const bool both = tshapes && sshapes, many = nrhs > 1;
  if ((long long)nt * ns < (both ? kSortedPairsBoth : kSortedPairs)) return false;
  const double step = both ? (many ? 20.0 : 17.0) : sshapes ? (many ? 13.0 : 6.05) : (many ? 8.5 : 5.6);
  const double rounds = nt / 16384.0, steps = nt <= 16384 ? 0.5 * cdiv(ns, 512)
                                                          : ns / 1024.0 * ((!both && many ? 0.95 : 0.8) * rounds + 0.7);
  double sorting = (tshapes ? 17.0 : 12.0) + sort_us(nt) + (same ? 0.0 : sort_us(ns)) + 2.5e-5 * nt * nrhs;
  if (both)  // the passes of eight columns keep few waves on a compute unit
    sorting += 2.5e-3 * std::min(nt, 16384) * (nrhs / 8 + (nrhs % 8 > 4 ? 1 : 0));
  return step * steps * cdiv(nrhs, 8) > sorting;
}

// For any of its shapes: those on both sides of one set ask for the most and are sorted
// wherever others are.
size_t gauss_pair_workspace(int nt, int ns, bool same, int nrhs) {
  if (nt <= 0 || ns <= 0 || nrhs <= 0 || !gauss_pair_sorted(nt, ns, true, true, true, nrhs)) return 0;
  Sizer s;
  TilePlan pt, ps;
  char* rest;
  size_t bytes;
  carve_pair(s, nt, ns, same, std::min(nrhs, 8), pt, ps, rest, bytes);
  return s.used;
}

static bool same_points(const GSide& T, const GSide& S) { return T.n == S.n && T.x == S.x && T.y == S.y; }

bool gauss_pair_sorted(const GSide& T, const GSide& S, int nrhs) {
  return gauss_pair_sorted(T.n, S.n, T.z != nullptr, S.z != nullptr, same_points(T, S), nrhs);
}

int gauss_pair_product(const GSide& T, const GSide& S, double base, double norm, int nrhs, const float* V, int ldv,
                       float* Y, int ldy, float beta, void* ws, size_t ws_bytes, hipStream_t stream,
                       const PlanSide* side) {
  const bool same = same_points(T, S);  // one set of points: one sort
  Carver cv(ws, ws_bytes);
  TilePlan pt, ps;
  char* rest;
  size_t bytes;
  carve_pair(cv, T.n, S.n, same, std::min(nrhs, 8), pt, ps, rest, bytes);
  if (!cv.ok()) return check_ws(ws, ws_bytes, gauss_pair_workspace(T.n, S.n, same, nrhs));
  GTileBufs b;
  GPL_TRY(gauss_tiles_carve(T.n, S.n, std::min(nrhs, 8), rest, bytes, b));
  GPL_TRY(plan_sort(pt, T.n, T.x, T.y, stream, side));
  if (!same) GPL_TRY(plan_sort(ps, S.n, S.x, S.y, stream));
  return gauss_tiles_product(sorted_view(pt), T.z, T.w, sorted_view(same ? pt : ps), S.z, S.w, base, norm, nrhs, V,
                             ldv, Y, ldy, beta, b, stream);
}

}  // namespace gpl
