// Conjugate gradients on a small image: an iteration in two launches, the kernel
// product and this file's kernel, instead of six. A workgroup holds one column of
// everything between two products in LDS: it adds up the column's partial rows
// (T = K B^T P), applies B, adds sigma^2 P and forms p.Ap; takes the step in X and R;
// takes the next direction P; and applies B^T to it, scaled, split and placed in the
// product's buffers. Every value is formed by the same operations in the same
// order as by the separate kernels (reduce_kernel, psf_forward_kernel,
// cg_update1/2_kernel, psf_adjoint_rhs_kernel), so the iterates have the same bits on
// either route: the taps of a composite filter in order, those outside the grid left
// out (they add exact zeros there), and the FP64 sums over the same threads of the
// same tiles and spans. (The batch of the serving loop runs the separate kernels; a test
// there asks for the same image bit for bit.)
//
// Bound by latency: six launches of some 4.5 us each do a microsecond's work apiece
// on up to 64 x 64 pixels. An iteration on 31 x 31 pixels and 4 columns takes 15.9 us
// instead of 30.9, 33 x 33 and 17 columns 20.2 for 32.2, 64 x 64 and 17 columns 30.6 for
// 35.4. Beyond 4,096 fine points the column's one compute unit is the slower way (48 x 48
// pixels twice supersampled, nine points a thread: 50.8 for 37.6). Its LDS leaves room for
// one workgroup on a compute unit, so more than 256 columns run in rounds: still no slower
// (a solve of 12 iterations, us for the separate kernels': 32 x 32 pixels 291 for 504 with 17
// columns, 594 for 836 with 256, 727 for 889 with 257, 1,965 for 2,087 with 1,024; 64 x 64
// 434 for 540, 921 for 1,129 and 1,180 for 1,223 with 17, 256 and 257).
#include <algorithm>
#include <cmath>

#include "cg_step.hpp"
#include "common.hpp"
#include "internal.hpp"

namespace gpl {

constexpr int kColThreads = 1024, kColGroups = kColThreads / 256;
constexpr int kColPix = 4096;   // pixels of the image: one span a group of 256 threads
constexpr int kColFine = 4096;  // fine points
constexpr int kColRows = 7424;  // floats of a padded window: 64 rows with 24 + 28 more at r = 24
constexpr int kColTiles = 64;   // output tiles of B, kColTile fine points a side
constexpr int kColTile = 32;
constexpr int kColTaps = 256;   // taps of B^T by phase
static_assert(kUpdSpan * kColGroups == kColPix, "a span a group");

static __host__ __device__ int col_tile_pixels(int ss) { return kColTile / ss > 0 ? kColTile / ss : 1; }

// Windows with their zeros. B: M rows of M + 2 r fine points, then M + 2 r rows of n
// pixels filtered along x. B^T: the pixels J + k, k < K4, with J = floor((f - r) / ss)
// reach fine point f with tap f + r - ss (J + k) (K4: their number, rounded up to
// whole fours): n rows of `lo` + n + `hi` pixels, then as many rows of M.
struct ColDims {
  int K4, lo, width;
};
static __host__ __device__ ColDims col_dims(int n, int ss, int r) {
  const int L = 2 * r + ss;
  ColDims d;
  d.K4 = ((L - 1) / ss + 4) / 4 * 4;
  d.lo = (r + ss - 1) / ss;
  const int last = (n * ss - 1 - r + 64 * ss) / ss - 64;  // J of the last fine point
  d.width = d.lo + max(n, last + d.K4);
  return d;
}

bool cg_column_fits(int n, int ss, int r) {
  const long M = (long)n * ss, npix = (long)n * n;
  const int tx = cdiv(n, col_tile_pixels(ss));
  if (npix > kColPix || M * M > kColFine || tx * tx > kColTiles || tx * tx != psf_forward_tiles(n, ss)) return false;
  const ColDims d = col_dims(n, ss, r);
  return M * (M + 2 * r) <= kColRows && (long)n * d.width <= kColRows && M * d.width <= kColRows &&
         ss * d.K4 <= kColTaps;
}

// floor(v / d) for 0 <= v < 2^16, d >= 1, rd = 1 / d in FP32 (d up to 64: (v + 1/2) / d
// stays 1/128 away from an integer, above the FP32 rounding of the product and of rd).
__device__ __forceinline__ int div_small(int v, float rd) { return (int)(((float)v + 0.5f) * rd); }

// out[q] = sum over k < K in order of w[k] in[at[q] + k step], `Q` outputs together.
template <int Q>
__device__ __forceinline__ void tap_sums(const float* w, const float* in, const int (&at)[Q], int step, int K,
                                         float (&out)[Q]) {
#pragma unroll
  for (int q = 0; q < Q; ++q) out[q] = 0.f;
  int k = 0;
#pragma unroll 1
  for (; k + 4 <= K; k += 4) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const float* p = in + at[q] + k * step;
      const float a = p[0], b = p[step], c = p[2 * step], d = p[3 * step];
      out[q] = fmaf(w[k], a, out[q]);
      out[q] = fmaf(w[k + 1], b, out[q]);
      out[q] = fmaf(w[k + 2], c, out[q]);
      out[q] = fmaf(w[k + 3], d, out[q]);
    }
  }
  for (; k < K; ++k)
#pragma unroll
    for (int q = 0; q < Q; ++q) out[q] = fmaf(w[k], in[at[q] + k * step], out[q]);
}
// The same, K a multiple of four, each output with its own taps.
template <int Q>
__device__ __forceinline__ void tap_sums_by(const float* w, const int (&wa)[Q], const float* in, const int (&at)[Q],
                                            int step, int K, float (&out)[Q]) {
#pragma unroll
  for (int q = 0; q < Q; ++q) out[q] = 0.f;
#pragma unroll 1
  for (int k = 0; k < K; k += 4) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const float4 g = *reinterpret_cast<const float4*>(w + wa[q] + k);
      const float* p = in + at[q] + k * step;
      const float a = p[0], b = p[step], c = p[2 * step], d = p[3 * step];
      out[q] = fmaf(g.x, a, out[q]);
      out[q] = fmaf(g.y, b, out[q]);
      out[q] = fmaf(g.z, c, out[q]);
      out[q] = fmaf(g.w, d, out[q]);
    }
  }
}

// OWN fine points (and entries of a window filtered along one axis) a thread.
template <int OWN>
__global__ __launch_bounds__(kColThreads) void cg_column_kernel(CgColumn C, const ColState* __restrict__ st_in,
                                                                ColState* __restrict__ st_out,
                                                                const int* __restrict__ active_in, int* active_out,
                                                                int* active_next) {
  __shared__ float win[kColRows];  // T in M rows; then the direction P in n rows
  __shared__ float mid[kColRows];  // either filtered along x
  __shared__ float ap[kColPix], pp[kColPix], tg[kMaxComposite];
  __shared__ __attribute__((aligned(16))) float tq[kColTaps];
  __shared__ double red[kColTiles][4];
  __shared__ float redm[kColGroups][4];
  __shared__ double s_alpha, s_beta;
  __shared__ int s_bad, s_go;
  const int tid = threadIdx.x, lane = tid & 63, t = tid & 255, wv = (tid >> 6) & 3, c = blockIdx.x;
  const int q = __builtin_amdgcn_readfirstlane(tid >> 8);
  const int n = C.n, ss = C.ss, M = n * ss, N = M * M, npix = n * n, r = C.taps.r, L = C.taps.L, W = M + 2 * r;
  const float rn = 1.f / (float)n, rM = 1.f / (float)M, rss = 1.f / (float)ss;
  const ColDims dim = col_dims(n, ss, r);
  const TilePlan& P = C.plan;
  // this thread's vector entries (span q), and the rows its fine points come from
  float xv[kUpdPer], pv[kUpdPer], rv[kUpdPer];
  int i[kUpdPer];
#pragma unroll
  for (int e = 0; e < kUpdPer; ++e) {
    i[e] = q * kUpdSpan + e * 256 + t;
    const int ic = min(i[e], npix - 1);
    xv[e] = C.X[(size_t)c * C.ldx + ic];
    pv[e] = C.P[(size_t)c * C.ldv + ic];
    rv[e] = C.R[(size_t)c * C.ldv + ic];
  }
  int2 sl[OWN];
  int dst[OWN], at[OWN];  // fine point of the thread's sorted positions, sorted position of its fine points
#pragma unroll
  for (int u = 0; u < OWN; ++u) {
    const int j = min(tid + u * kColThreads, N - 1);
    sl[u] = P.rslot[j / kRowTile];
    dst[u] = P.perm[j];
    at[u] = C.rhs.irank[j];
  }
  const ColState st = st_in[c];
  if (c == 0 && tid == 0) *active_next = 0;
  if (*active_in == 0 || !st.active) {  // carry the state into the other parity
    if (tid == 0) st_out[c] = st;
    return;
  }
#pragma unroll
  for (int e = 0; e < kUpdPer; ++e)
    if (i[e] < npix) pp[i[e]] = pv[e];
  if (tid < L) tg[tid] = C.taps.g[tid];
  for (int k = tid; k < ss * dim.K4; k += kColThreads) {
    const int ph = k / dim.K4, tap = ph + 2 * r - ss * (k - ph * dim.K4);
    tq[k] = tap >= 0 && tap < L ? C.taps.g[tap] : 0.f;
  }
  for (int k = tid; k < M * W; k += kColThreads) win[k] = 0.f;
  for (int k = tid; k < W * n; k += kColThreads) mid[k] = 0.f;
  // T of this column: the partial rows in slot order
  float T[OWN] = {};
  {
    const size_t stride = (size_t)C.nrhs * kRowTile;
    const float* base = C.bufs.part + (size_t)c * kRowTile;
    const float cs = C.bufs.inv_scale ? C.bufs.inv_scale[c] : 1.f;
    const float* p0[OWN];
    int cnt = 0;
#pragma unroll
    for (int u = 0; u < OWN; ++u) {
      p0[u] = base + (size_t)sl[u].x * stride + ((tid + u * kColThreads) & (kRowTile - 1));
      cnt = max(cnt, sl[u].y);
    }
    for (int s0 = 0; s0 < cnt; s0 += 8) {
      float v[OWN][8];
#pragma unroll
      for (int u = 0; u < OWN; ++u)
#pragma unroll
        for (int k = 0; k < 8; ++k) v[u][k] = p0[u][(size_t)max(min(s0 + k, sl[u].y - 1), 0) * stride];
#pragma unroll
      for (int u = 0; u < OWN; ++u)
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (s0 + k < sl[u].y) T[u] += v[u][k];
    }
#pragma unroll
    for (int u = 0; u < OWN; ++u) {
      const float as = C.amp2 * T[u];
      T[u] = C.bufs.inv_scale ? as * cs : as;
    }
  }
  __syncthreads();  // the windows are clear
#pragma unroll
  for (int u = 0; u < OWN; ++u)
    if (tid + u * kColThreads < N) {
      const int y = div_small(dst[u], rM);
      win[y * W + r + dst[u] - y * M] = T[u];
    }
  __syncthreads();
  // B along x, then along y
  {
    int from[OWN], to[OWN];
    float v[OWN];
#pragma unroll
    for (int u = 0; u < OWN; ++u) {
      const int o = min(tid + u * kColThreads, M * n - 1), y = div_small(o, rn);
      from[u] = y * W + ss * (o - y * n);
      to[u] = o + r * n;
    }
    tap_sums<OWN>(tg, win, from, 1, L, v);
#pragma unroll
    for (int u = 0; u < OWN; ++u)
      if (tid + u * kColThreads < M * n) mid[to[u]] = v[u];
  }
  __syncthreads();
  const int TP = col_tile_pixels(ss), tiles_x = cdiv(n, TP);
  const float inv_ss2 = 1.f / (float)(ss * ss);
  const float rTP = 1.f / (float)TP;
  for (int tile = q; tile < C.ntiles; tile += kColGroups) {
    const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
    double dot = 0.0;
    constexpr int kPer = kColTile * kColTile / 256;
    int I[kPer], from[kPer];
    float v[kPer];
    const int per = cdiv(TP * TP, 256);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int o = t + u * 256, oy = div_small(o, rTP), Iy = ty * TP + oy, Ix = tx * TP + o - oy * TP;
      I[u] = o < TP * TP && Iy < n && Ix < n ? Iy * n + Ix : -1;
      from[u] = I[u] < 0 ? 0 : ss * Iy * n + Ix;
    }
    if (per > 1) {
      tap_sums<kPer>(tg, mid, from, n, L, v);
    } else {
      int one[1] = {from[0]};
      float w[1];
      tap_sums<1>(tg, mid, one, n, L, w);
      v[0] = w[0];
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u)
      if (I[u] >= 0) {
        const float p = pp[I[u]], res = fmaf(C.sigma2, p, v[u] * inv_ss2);
        ap[I[u]] = res;
        dot += (double)p * (double)res;
      }
    dot = warp_sum(dot);
    if (lane == 0) red[tile][wv] = dot;
  }
  __syncthreads();
  if (tid < 64) {
    double s = 0.0;
    if (lane < C.ntiles) {
#pragma unroll
      for (int w = 0; w < 4; ++w) s += red[lane][w];
    }
    const double pap = warp_sum(s);
    if (lane == 0) {
      const ColumnAlpha a = cg_alpha(st.rr, pap);
      s_alpha = a.alpha;
      s_bad = a.bad;
    }
  }
  __syncthreads();
  // the step; T and its filtered rows have been read
  for (int k = tid; k < n * dim.width; k += kColThreads) win[k] = 0.f;
  for (int k = tid; k < dim.width * M; k += kColThreads) mid[k] = 0.f;
  {
    double s = 0.0;
    if (!s_bad) {
      const float af = (float)s_alpha;
#pragma unroll
      for (int e = 0; e < kUpdPer; ++e)
        if (i[e] < npix) {
          C.X[(size_t)c * C.ldx + i[e]] = fmaf(af, pv[e], xv[e]);
          rv[e] = fmaf(-af, ap[i[e]], rv[e]);
          C.R[(size_t)c * C.ldv + i[e]] = rv[e];
          s += (double)rv[e] * rv[e];
        }
    }
    s = warp_sum(s);
    if (lane == 0) red[q][wv] = s;
  }
  __syncthreads();
  if (tid < 64) {
    double s = 0.0;
    if (lane < cdiv(npix, kUpdSpan)) {
#pragma unroll
      for (int w = 0; w < 4; ++w) s += red[lane][w];
    }
    const double rr_new = warp_sum(s);
    if (lane == 0) {
      const ColumnStep k = cg_step(st, s_alpha, s_bad, rr_new, c, C.bb, C.tol, C.max_iter, C.fixed_iters, C.n_lanczos,
                                   C.ab, true);
      s_beta = k.beta;
      s_go = k.go;
      st_out[c] = k.next;
      if (k.next.active) atomicAdd(active_out, 1);
    }
  }
  __syncthreads();
  if (!s_go) return;
  // the next direction and the scale of its B^T P
  {
    const float bf = (float)s_beta;
    float m = 0.f;
#pragma unroll
    for (int e = 0; e < kUpdPer; ++e)
      if (i[e] < npix) {
        const float pn = fmaf(bf, pv[e], rv[e]);
        C.P[(size_t)c * C.ldv + i[e]] = pn;
        const int y = div_small(i[e], rn);
        win[y * dim.width + dim.lo + i[e] - y * n] = pn;
        m = fmaxf(m, fabsf(pn));
      }
    m = warp_max(m);
    if (lane == 0) redm[q][wv] = m;
  }
  __syncthreads();
  float scale = 1.f;
  const bool f16 = C.rhs.prec == GPL_PREC_F16X3;
  if (f16) {
    float m = 0.f;
#pragma unroll
    for (int g = 0; g < kColGroups; ++g)
#pragma unroll
      for (int w = 0; w < 4; ++w) m = fmaxf(m, redm[g][w]);
    const float mx = m / (float)(ss * ss);
    int e = 0;
    if (mx > 0.f && isfinite(mx)) e = min(14 - ilogbf(mx) - 1, 126);
    scale = ldexpf(1.f, e);
    if (tid == 0) C.rhs.inv_scale[c] = ldexpf(1.f, -e) / 2048.f;
  }
  // B^T along x, then along y
  auto first = [&](int f) { return div_small(f - r + 64 * ss, rss) - 64; };  // J of fine point f
  {
    int from[OWN], wa[OWN], to[OWN];
    float v[OWN];
#pragma unroll
    for (int u = 0; u < OWN; ++u) {
      const int o = min(tid + u * kColThreads, n * M - 1), y = div_small(o, rM), f = o - y * M, J = first(f);
      from[u] = y * dim.width + dim.lo + J;
      wa[u] = (f - r - ss * J) * dim.K4;
      to[u] = o + dim.lo * M;
    }
    tap_sums_by<OWN>(tq, wa, win, from, 1, dim.K4, v);
#pragma unroll
    for (int u = 0; u < OWN; ++u)
      if (tid + u * kColThreads < n * M) mid[to[u]] = v[u];
  }
  __syncthreads();
  const int hs = hi_slot(c, C.rhs.nrhs), ncp = C.rhs.ncp;
  const bool packed = last_block_packed(C.rhs.nrhs) && c >= packed_block_start(C.rhs.nrhs);
  int from[OWN], wa[OWN];
  float v[OWN];
#pragma unroll
  for (int u = 0; u < OWN; ++u) {
    const int o = min(tid + u * kColThreads, N - 1), f = div_small(o, rM), J = first(f);
    from[u] = (dim.lo + J) * M + o - f * M;
    wa[u] = (f - r - ss * J) * dim.K4;
  }
  tap_sums_by<OWN>(tq, wa, mid, from, M, dim.K4, v);
#pragma unroll
  for (int u = 0; u < OWN; ++u) {
    if (tid + u * kColThreads >= N) break;
    const float b = v[u] * inv_ss2;
    if (f16) {
      const size_t j = rhs_at(hs, at[u], ncp);
      const float sv = b * scale;
      const _Float16 h = (_Float16)sv, l = (_Float16)(sv - (float)h);
      C.rhs.Vh[j] = h;
      if (packed) C.rhs.Vh[j + kChunk] = l;  // slot hs + 1 of the same chunk
      else C.rhs.Vl[j] = l;
    } else {
      C.rhs.Vp[rhs_at(c, at[u], ncp)] = b;
    }
  }
}

int cg_column_launch(const CgColumn& C, const ColState* st_in, ColState* st_out, const int* active_in, int* active_out,
                     int* active_next, hipStream_t stream) {
  GPL_REQUIRE(cg_column_fits(C.n, C.ss, C.taps.r), "image too large for a workgroup");
  static_assert(kColFine == 4 * kColThreads, "one, two or four points a thread");
  const int N = C.n * C.ss * C.n * C.ss;
  const auto kern = N <= kColThreads       ? cg_column_kernel<1>
                    : N <= 2 * kColThreads ? cg_column_kernel<2>
                                           : cg_column_kernel<4>;
  hipLaunchKernelGGL(kern, dim3(C.nrhs), dim3(kColThreads), 0, stream, C, st_in, st_out, active_in,
                     active_out, active_next);
  GPL_LAUNCH_CHECK();
  return GPL_OK;
}

}  // namespace gpl
