// Distance to the k-th closest other point, for the density of inducing points
// of the transmission weights (Sec. 3.4, footnote to eq. "transmission": the
// area of the circle reaching the k-th closest point, k = 20).
//
// The points are sorted along the Hilbert curve of the tile plan and grouped in
// 32-point chunks with bounding boxes. One wave takes one point: its lanes hold
// 64 candidates at a time, and those that beat the current bound on the k-th
// key are appended to a buffer in LDS. When more than 64 are held, the k
// smallest are selected (by counting below a pivot with ballots) and the k-th
// becomes the bound. The point's own 64-point tile and its two neighbours along
// the curve come first; then the boxes of all chunks are tested against the
// bound, 64 at a time, and only the chunks within reach are visited, two at a
// time. Keys are (squared distance in FP32, caller index) in one 64-bit
// integer, so equal distances rank the lower index first.
//
// Bound by latency and issue: about 20 box tests, 10 visits and 3 selections a
// point at 40,000 points. A lane per point with a sorted list in registers (a
// serial insertion through 32 slots per accepted candidate, and 625 waves for
// 40,000 points) took 800 us at 40,000 traced points and 590 us at 1600.
#include <climits>
#include <cmath>

#include "common.hpp"
#include "internal.hpp"
#include "tileplan.hpp"

namespace gpl {

constexpr int kKnnMaxK = 32;
constexpr int kKnnWaves = 4;                // points (waves) per workgroup
constexpr int kKnnBuf = 128;                // candidates held: at most 64 kept and 64 new
constexpr int kKnnBoxes = 4;                // box tests of a lane in flight
static_assert(kKnnMaxK <= 64, "the kept candidates fit the first half of the buffer");

using KnnKey = unsigned long long;
constexpr KnnKey kKnnNone = (0x7f800000ull << 32) | (KnnKey)INT_MAX;  // no k-th neighbour yet: (inf, INT_MAX)

__device__ __forceinline__ int mask_rank(unsigned long long m) {  // set bits of m below this lane
  return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

__device__ __forceinline__ KnnKey lane_key(KnnKey v, int lane) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), lane);
  return ((KnnKey)hi << 32) | lo;
}

// k-th smallest (1-based) of the wave's keys: a in the lanes of ma, b in those
// of mb, all distinct, at least k of them. Quickselect: each round drops the
// pivot's side that cannot hold the answer, so it ends after at most as many
// rounds as there are keys.
__device__ __forceinline__ KnnKey wave_select(KnnKey a, KnnKey b, unsigned long long ma, unsigned long long mb, int k) {
  while (true) {
    const KnnKey p = ma ? lane_key(a, __ffsll((long long)ma) - 1) : lane_key(b, __ffsll((long long)mb) - 1);
    const unsigned long long la = __ballot(a < p) & ma, lb = __ballot(b < p) & mb;
    const int below = __popcll(la) + __popcll(lb);
    if (below == k - 1) return p;
    if (below >= k) {
      ma = la;
      mb = lb;
    } else {
      k -= below + 1;
      ma &= ~la & __ballot(a != p);
      mb &= ~lb & __ballot(b != p);
    }
  }
}

__device__ __forceinline__ unsigned long long low_mask(int n) { return n >= 64 ? ~0ull : (1ull << n) - 1ull; }

// A set of sorted points and its outputs; the workgroups from `block0` on are its.
struct KnnArgs {
  int n, nch, block0;
  const float *xs, *ys;
  const int* perm;
  const float4* cbox;
  float *rho, *rk, *w;
  int* nn;
};

__global__ __launch_bounds__(64 * kKnnWaves) void knn_sorted_kernel(KnnArgs first, KnnArgs second, int k, float scale) {
  __shared__ KnnKey sbuf[kKnnWaves][kKnnBuf];
  const KnnArgs& S = (int)blockIdx.x < second.block0 ? first : second;
  const int n = S.n, nch = S.nch;
  const float *__restrict__ xs = S.xs, *__restrict__ ys = S.ys;
  const int* __restrict__ perm = S.perm;
  const float4* __restrict__ cbox = S.cbox;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int i = ((int)blockIdx.x - S.block0) * kKnnWaves + wv;  // sorted position of the wave's point
  if (i >= n) return;                                           // whole waves leave; no workgroup barrier below
  KnnKey* buf = sbuf[wv];
  const float xi = xs[i], yi = ys[i];
  const int me = perm[i];
  KnnKey bound = kKnnNone;  // only keys below it can be among the k smallest
  int cnt = 0;              // keys held in buf
  auto keys = [&](KnnKey& a, KnnKey& b) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    a = buf[lane];  // entries past cnt are masked out by the caller
    b = buf[64 + lane];
  };
  auto shrink = [&] {
    KnnKey a, b;
    keys(a, b);
    unsigned long long ma = low_mask(cnt), mb = low_mask(max(cnt - 64, 0));
    bound = wave_select(a, b, ma, mb, k);
    ma &= __ballot(a <= bound);
    mb &= __ballot(b <= bound);
    const int na = __popcll(ma);
    if ((ma >> lane) & 1ull) buf[mask_rank(ma)] = a;
    if ((mb >> lane) & 1ull) buf[na + mask_rank(mb)] = b;
    cnt = k;
  };
  auto visit = [&](int ca, int cb) {  // chunk ca in the lower lanes, cb (-1: none) in the upper
    const int c = lane < 32 ? ca : cb;
    const int j = c * kChunk + (lane & 31);
    bool ok = c >= 0 && j < n;
    const int jj = ok ? j : i;
    const float dx = xi - xs[jj], dy = yi - ys[jj];
    const int id = perm[jj];
    const float d2 = fmaf(dx, dx, dy * dy);
    const KnnKey key = ((KnnKey)__float_as_uint(d2) << 32) | (unsigned)id;  // a NaN ranks above kKnnNone
    ok = ok && id != me && key < bound;
    const unsigned long long m = __ballot(ok);
    if (m == 0ull) return;
    if (ok) buf[cnt + mask_rank(m)] = key;
    cnt += __popcll(m);
    if (cnt > 64) shrink();
  };
  static_assert(kChunk == 32, "two chunks fill a wave");
  const int own = i / kRowTile * kChunksPerTile;  // first chunk of the point's tile
  const int lo = max(0, own - kChunksPerTile), hi = min(nch, own + 2 * kChunksPerTile);
  visit(own, own + 1);
  if (lo < own) visit(lo, lo + 1);
  if (own + kChunksPerTile < hi) visit(own + kChunksPerTile, own + kChunksPerTile + 1);
  if (cnt > k) shrink();
  for (int c0 = 0; c0 < nch; c0 += 64 * kKnnBoxes) {
    float4 q[kKnnBoxes];
#pragma unroll
    for (int u = 0; u < kKnnBoxes; ++u) q[u] = cbox[min(c0 + 64 * u + lane, nch - 1)];
#pragma unroll
    for (int u = 0; u < kKnnBoxes; ++u) {
      const int c = c0 + 64 * u + lane;
      const float gx = fmaxf(0.f, fmaxf(q[u].x - xi, xi - q[u].y));
      const float gy = fmaxf(0.f, fmaxf(q[u].z - yi, yi - q[u].w));
      // the gap is at most the FP32 distance of any point of the chunk
      const bool need = c < nch && !(c >= lo && c < hi) &&
                        fmaf(gx, gx, gy * gy) <= __uint_as_float((unsigned)(bound >> 32));
      unsigned long long m = __ballot(need);
      while (m != 0ull) {
        const int a = __ffsll((long long)m) - 1;
        m &= m - 1ull;
        const int b = m ? __ffsll((long long)m) - 1 : -1;
        m &= m ? m - 1ull : 0ull;
        visit(c0 + 64 * u + a, b < 0 ? -1 : c0 + 64 * u + b);
      }
    }
  }
  KnnKey kth = kKnnNone;
  if (cnt >= k) {
    KnnKey a, b;
    keys(a, b);
    kth = wave_select(a, b, low_mask(cnt), low_mask(max(cnt - 64, 0)), k);
  }
  if (lane != 0) return;
  const float d2 = __uint_as_float((unsigned)(kth >> 32));
  if (S.rho) S.rho[me] = (float)k / ((float)M_PI * d2);
  if (S.rk) S.rk[me] = sqrtf(d2);
  if (S.w) S.w[me] = scale * sqrtf(d2);
  if (S.nn) S.nn[me] = kth == kKnnNone ? -1 : (int)(unsigned)kth;  // -1: fewer than k comparable points
}

static size_t knn_workspace(int n) {
  Sizer s;
  TilePlan p;
  sort_carve(s, n, p);
  return s.used;
}

static int check_knn(int n, int k) {
  GPL_REQUIRE(k >= 1 && k <= kKnnMaxK && n > k, "k=%d must be in [1, %d] and below n=%d", k, kKnnMaxK, n);
  GPL_REQUIRE(n <= kMaxPlanChunks * kChunk, "n=%d exceeds the limit of %d points", n, kMaxPlanChunks * kChunk);
  return GPL_OK;
}

int knn_sorted_launch(const KnnSet* sets, int nsets, int k, float scale, hipStream_t stream) {
  KnnArgs a[2] = {};
  int blocks = 0;
  for (int q = 0; q < 2; ++q) {
    a[q].block0 = blocks;
    if (q >= nsets) continue;
    const TilePlan& p = sets[q].plan;
    GPL_TRY(check_knn(p.n, k));
    a[q] = KnnArgs{p.n, p.nch, blocks, p.xs, p.ys, p.perm, p.cbox, sets[q].rho, sets[q].rk, sets[q].w, sets[q].nn};
    blocks += cdiv(p.n, kKnnWaves);
  }
  hipLaunchKernelGGL(knn_sorted_kernel, dim3(blocks), dim3(64 * kKnnWaves), 0, stream, a[0], a[1], k, scale);
  GPL_LAUNCH_CHECK();
  return GPL_OK;
}

}  // namespace gpl

using namespace gpl;

extern "C" size_t gpl_knn_density_workspace(int n) { return n <= 0 ? 0 : knn_workspace(n); }

extern "C" int gpl_knn_density(int n, const float* qx, const float* qy, int k, float* rho, void* ws, size_t ws_bytes,
                               hipStream_t stream) {
  GPL_REQUIRE(qx && qy && rho, "NULL argument");
  GPL_TRY(check_knn(n, k));
  GPL_TRY(check_ws(ws, ws_bytes, knn_workspace(n)));
  Carver cv(ws, ws_bytes);
  TilePlan p;
  sort_carve(cv, n, p);
  if (!cv.ok()) return check_ws(nullptr, 0, 1);
  GPL_TRY(plan_sort(p, n, qx, qy, stream));
  const KnnSet set{p, rho, nullptr, nullptr, nullptr};
  return knn_sorted_launch(&set, 1, k, 0.f, stream);
}
