// Construction of the tile plan of the kernel product (see tileplan.hpp): sorted
// points, chunk bounding boxes, and per row tile the list of chunks within the
// exact-zero cutoff of the kernel (Sec. 3.1, eq. "grbf").
//
// A plan is built for every product that is not part of a solve, so its launches
// count as much as the product itself: every kernel of it is bound by latency.
// Nine launches (one up to kSmallPoints points) instead of twenty-two: two sort
// passes of 12 bits in which each workgroup folds all workgroups' digit counts
// itself (no scan launches between), boxes and scaled coordinates in one kernel,
// and the split over the waves in two.
#include <cmath>
#include <type_traits>
#include <utility>

#include "mvm_rhs.hpp"
#include "tile_boxes.hpp"
#include "tileplan.hpp"

namespace gpl {

size_t plan_workspace(int n) {
  if (n <= 0) return 0;
  Sizer s;
  TilePlan p;
  plan_carve(s, n, p);
  return s.used;
}

// ---- point order: Hilbert keys, then a stable LSD radix sort ----

// Four-way extent (xmin, xmax, ymin, ymax) over the lanes of a wave.
__device__ __forceinline__ float4 wave_extent(float4 e) {
  e = join_lane_xor<8>(e);
  e = join_lane_xor<4>(e);
  e = join_lane_xor<2>(e);
  e = join_lane_xor<1>(e);
  e = join_lane_xor<16>(e);
  return join_lane_xor<32>(e);
}

// Extent of the finite points among first, first + step, ... below n for this
// thread; 4 points a round, their loads issued together (an index past n reads
// point 0 and is not used).
__device__ __forceinline__ float4 thread_extent(int n, const float* __restrict__ px, const float* __restrict__ py,
                                                int first, int step) {
  float4 e = make_float4(kInf, -kInf, kInf, -kInf);
  constexpr int kU = 4;
  for (int i0 = first; i0 < n; i0 += kU * step) {
    float x[kU], y[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int i = i0 + u * step < n && i0 + u * step >= 0 ? i0 + u * step : 0;
      x[u] = px[i];
      y[u] = py[i];
    }
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (i0 + u * step < n && isfinite(x[u]) && isfinite(y[u]))
        e = join_extent(e, make_float4(x[u], x[u], y[u], y[u]));
  }
  return e;
}

// (xmin, ymin, side of the square from there that holds every finite point, 0).
__device__ __forceinline__ float4 extent_square(const float4& e) {
  if (!(e.x <= e.y)) return make_float4(0.f, 0.f, 0.f, 0.f);  // no finite point
  return make_float4(e.x, e.z, fmaxf(e.y - e.x, e.w - e.z), 0.f);
}

// Partial extents, one per workgroup (at most 64: the key kernel folds them).
__device__ __forceinline__ void extent_part(int n, const float* __restrict__ px, const float* __restrict__ py,
                                            int parts, float4* part) {
  __shared__ float4 red[kSortThreads / 64];
  float4 e = wave_extent(thread_extent(n, px, py, blockIdx.x * kSortThreads + threadIdx.x, parts * kSortThreads));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = e;
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int k = 1; k < kSortThreads / 64; ++k) e = join_extent(e, red[k]);
  part[blockIdx.x] = e;
}

__global__ __launch_bounds__(kSortThreads) void plan_extent_kernel(int n, const float* __restrict__ px,
                                                                   const float* __restrict__ py, float4* part) {
  extent_part(n, px, py, gridDim.x, part);
}

// The right-hand sides of a product that follows the plan are prepared beside it: the
// column maxima with the extent, their places in the sorted order with the last
// kernel of the plan, a single workgroup. In launches of their own these took 4.0 and
// 5.0 us at 40,000 points and 17 columns, 10 and 29 at 160,000 and 64; the product
// takes 93.7 us for 102 with them there, and 281 for 299.
__global__ __launch_bounds__(kSortThreads) void plan_extent_rhs_kernel(int n, const float* __restrict__ px,
                                                                       const float* __restrict__ py, int parts,
                                                                       float4* part, RhsJob J) {
  __shared__ float red[kSortThreads / 64];
  if ((int)blockIdx.x < parts) {
    extent_part(n, px, py, parts, part);
  } else {
    const int g = threadIdx.x >> 8;
    colmax_unit(J, ((int)blockIdx.x - parts) * (kSortThreads / 256) + g, threadIdx.x & 255, red + 4 * g);
  }
}

// Index of cell (x, y) along the Hilbert curve of a 2^kHilbertBits square grid:
// at each level the quadrant contributes its position along the curve's U
// (0 lower left, 1 upper left, 2 upper right, 3 lower right), and the cell is
// mapped into the frame of that quadrant's copy of the curve.
__device__ __forceinline__ uint32_t hilbert_index(uint32_t x, uint32_t y) {
  constexpr uint32_t side = 1u << kHilbertBits;
  uint32_t d = 0;
  for (uint32_t s = side >> 1; s > 0; s >>= 1) {
    const uint32_t rx = (x & s) ? 1u : 0u, ry = (y & s) ? 1u : 0u;
    d += s * s * ((3u * rx) ^ ry);
    if (ry == 0) {
      if (rx == 1) {
        x ^= side - 1;
        y ^= side - 1;
      }
      const uint32_t t = x;
      x = y;
      y = t;
    }
  }
  return d;
}

// Sort key of a point: its Hilbert index on the grid over the extent; a point
// with a non-finite coordinate takes the last key.
__device__ __forceinline__ uint32_t point_key(float x, float y, const float4& e) {
  constexpr float kMaxCell = (float)((1u << kHilbertBits) - 1);
  if (!(isfinite(x) && isfinite(y))) return (1u << (2 * kHilbertBits)) - 1;
  const float sc = e.z > 0.f ? (float)(1u << kHilbertBits) / e.z : 0.f;
  const float qx = fminf(fmaxf((x - e.x) * sc, 0.f), kMaxCell);
  const float qy = fminf(fmaxf((y - e.y) * sc, 0.f), kMaxCell);
  return hilbert_index((uint32_t)qx, (uint32_t)qy);
}
__device__ __forceinline__ int key_digit(uint32_t k, int pass) {
  return (int)((k >> (kSortBits * pass)) & (kSortDigits - 1));
}

// The digit counts of a workgroup's items, h in LDS: cleared, counted by the
// caller between the two calls, then written as one row of hist.
__device__ __forceinline__ void clear_counts(int* h) {
  for (int d = threadIdx.x; d < kSortDigits; d += kSortThreads) h[d] = 0;
  __syncthreads();
}
__device__ __forceinline__ void store_counts(const int* h, SortCount* __restrict__ row) {
  __syncthreads();
  for (int d = threadIdx.x; d < kSortDigits; d += kSortThreads) row[d] = (SortCount)h[d];
}

// Keys of every point and the counts of their low digit: workgroup b takes the
// items [b span, (b + 1) span).
__global__ __launch_bounds__(kSortThreads) void plan_keys_kernel(int n, int span, const float* __restrict__ px,
                                                                 const float* __restrict__ py,
                                                                 const float4* __restrict__ part, int nparts,
                                                                 uint32_t* __restrict__ key,
                                                                 SortCount* __restrict__ hist) {
  __shared__ int h[kSortDigits];
  __shared__ float4 ext;
  if (threadIdx.x < 64) {
    const float4 e = wave_extent(part[min((int)threadIdx.x, nparts - 1)]);
    if (threadIdx.x == 0) ext = extent_square(e);
  }
  clear_counts(h);
  const float4 e = ext;
  const int end = min(n, ((int)blockIdx.x + 1) * span);
  for (int i = blockIdx.x * span + threadIdx.x; i < end; i += kSortThreads) {
    const uint32_t k = point_key(px[i], py[i], e);
    key[i] = k;
    atomicAdd(&h[key_digit(k, 0)], 1);
  }
  store_counts(h, hist + (size_t)blockIdx.x * kSortDigits);
}

// Counts of a later digit, the items in the order of the pass before.
__global__ __launch_bounds__(kSortThreads) void sort_count_kernel(int n, int span, int pass,
                                                                  const uint32_t* __restrict__ key,
                                                                  SortCount* __restrict__ hist) {
  __shared__ int h[kSortDigits];
  clear_counts(h);
  const int end = min(n, ((int)blockIdx.x + 1) * span);
  for (int i = blockIdx.x * span + threadIdx.x; i < end; i += kSortThreads) atomicAdd(&h[key_digit(key[i], pass)], 1);
  store_counts(h, hist + (size_t)blockIdx.x * kSortDigits);
}

// Exclusive prefix of one int per thread of the workgroup; ws: a wave's sums.
__device__ __forceinline__ int block_exclusive(int v, int* ws) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int x = warp_prefix(v);
  if (lane == 63) ws[w] = x;
  __syncthreads();
  int before = 0;
#pragma unroll
  for (int k = 0; k < kSortThreads / 64; ++k) before += k < w ? ws[k] : 0;
  return before + x - v;
}

// Stable ranking of one item per thread: the items of waves 0, 1, ... in turn,
// those of a wave by lane. pos[d] (LDS) is the next free position of digit d, wcnt[d]
// holds a byte per wave, the wave's items of the digit; all zero before and after. The
// lanes that hold the same digit find each other by ballots; the first of them
// writes the count and adds up the bytes of the waves before. (A turn of the workgroup
// per wave, each adding to pos in its turn, took 2.0 of a scatter's 14.5 us at 40,000
// points.) Returns the item's position (valid items only); more: another round follows.
static_assert(kSortThreads == 16 * 64, "a byte of a uint4 per wave");
__device__ __forceinline__ int rank_items(int d, bool valid, bool more, int* pos, uint4* wcnt) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  unsigned long long m = __ballot(valid);
#pragma unroll
  for (int b = 0; b < kSortBits; ++b) {
    const bool bit = (d >> b) & 1;
    const unsigned long long bb = __ballot(bit);
    m &= bit ? bb : ~bb;
  }
  const int lower = __popcll(m & ((1ull << lane) - 1ull)), first = valid ? __ffsll((long long)m) - 1 : 0;
  const bool leads = valid && lower == 0;
  unsigned char* mine = reinterpret_cast<unsigned char*>(wcnt + d) + w;
  if (leads) *mine = (unsigned char)__popcll(m);
  __syncthreads();
  int p = 0;
  bool last = false;
  if (leads) {
    const uint4 c = wcnt[d];
    const uint32_t cw[4] = {c.x, c.y, c.z, c.w};
    uint32_t sum = 0u, after = 0u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int bits = min(max(8 * (w - 4 * k), 0), 32);  // the bytes of the waves before this one
      const uint32_t below = bits == 32 ? ~0u : (1u << bits) - 1u;
      const uint32_t here = bits == 32 || w < 4 * k ? 0u : 0xffu << bits;
      sum = __builtin_amdgcn_sad_u8(cw[k] & below, 0u, sum);
      after |= cw[k] & ~(below | here);
    }
    p = pos[d] + (int)sum;
    last = after == 0u;
  }
  const int r = __shfl(p, first, 64) + lower;
  if (more) {
    __syncthreads();
    if (leads) {
      if (last) pos[d] = p + __popcll(m);
      *mine = 0;
    }
    __syncthreads();
  }
  return r;
}

// First position of every digit for a workgroup's items, into pos: the digits below,
// and the items of the digit in the workgroups before blk (hist: a row of counts per
// workgroup). Bound by latency and issue, few workgroups run: so one sweep over the
// rows, a thread taking eight digits of every other row with kFold loads in flight,
// the counts of a round added in 16 bits (at most 65,535 items) and the rounds in 32.
// (Four digits a thread, rows before and after in sweeps of their own, took 4.7 us of
// a scatter's 14.5 at 40,000 points; with the ranking above the first scatter takes
// 9.6 us instead of 14.5 and the last 12.6 instead of 16.4, at 160,000 18.0 instead of
// 22.4 and 26.8 instead of 30.6.) tmp: 16 kSortThreads / 2 ints.
__device__ __forceinline__ void digit_positions(const SortCount* __restrict__ hist, int blk, int nb, int span, int* pos,
                                                int* tmp, int* ws) {
  constexpr int kFold = 20, kHalf = kSortThreads / 2;
  static_assert(kSortDigits == 8 * kHalf, "eight digits of a row per thread");
  const int half = __builtin_amdgcn_readfirstlane(threadIdx.x / kHalf), g = threadIdx.x % kHalf;
  const uint4* row = reinterpret_cast<const uint4*>(hist) + g;
  const int per = min(kFold, 65535 / span);  // rows of a round
  int all[8], bef[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) all[k] = bef[k] = 0;
  for (int b0 = half; b0 < nb; b0 += 2 * per) {
    uint4 v[kFold];
#pragma unroll
    for (int u = 0; u < kFold; ++u) v[u] = row[(size_t)min(b0 + 2 * u, nb - 1) * (kSortDigits / 8)];
    uint4 a = make_uint4(0u, 0u, 0u, 0u), b = a;
#pragma unroll
    for (int u = 0; u < kFold; ++u) {
      const int r = b0 + 2 * u;
      const uint32_t live = u < per && r < nb ? ~0u : 0u, before = u < per && r < blk ? ~0u : 0u;
      a.x += v[u].x & live, a.y += v[u].y & live, a.z += v[u].z & live, a.w += v[u].w & live;
      b.x += v[u].x & before, b.y += v[u].y & before, b.z += v[u].z & before, b.w += v[u].w & before;
    }
    const uint32_t ap[4] = {a.x, a.y, a.z, a.w}, bp[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      all[2 * k] += (int)(ap[k] & 0xffffu), all[2 * k + 1] += (int)(ap[k] >> 16);
      bef[2 * k] += (int)(bp[k] & 0xffffu), bef[2 * k + 1] += (int)(bp[k] >> 16);
    }
  }
  if (half == 1)
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      tmp[k * kHalf + g] = all[k];
      tmp[(8 + k) * kHalf + g] = bef[k];
    }
  __syncthreads();
  int sum = 0;
  if (half == 0)
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      all[k] += tmp[k * kHalf + g];
      bef[k] += tmp[(8 + k) * kHalf + g];
      sum += all[k];
    }
  int run = block_exclusive(sum, ws);
  if (half == 0) {
    int p[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      p[k] = run + bef[k];
      run += all[k];
    }
    int4* out = reinterpret_cast<int4*>(pos + 8 * g);
    out[0] = make_int4(p[0], p[1], p[2], p[3]);
    out[1] = make_int4(p[4], p[5], p[6], p[7]);
  }
}

// Stable scatter of one pass. Every workgroup folds the counts of all workgroups
// (hist, one row each) into the first position of each digit for its own items.
// The last pass writes the sorted points instead of keys.
struct ScatterLds {
  __attribute__((aligned(16))) int pos[kSortDigits];
  uint4 wcnt[kSortDigits];
};
template <bool kLast>
__device__ __forceinline__ void sort_scatter_body(ScatterLds& L, int nb, int n, int span, int pass,
                                                  const uint32_t* __restrict__ kin, const int* __restrict__ vin,
                                                  const SortCount* __restrict__ hist,
                                                  uint32_t* __restrict__ kout, int* __restrict__ vout,
                                                  const float* __restrict__ px, const float* __restrict__ py,
                                                  int* __restrict__ irank, float* __restrict__ xs,
                                                  float* __restrict__ ys) {
  __shared__ int wsum[kSortThreads / 64];
  int* const pos = L.pos;
  uint4* const wcnt = L.wcnt;
  const int blk = blockIdx.x;
  const int end = min(n, (blk + 1) * span);
  // an item's key and index, and in the last pass its point: loaded ahead of the
  // work they do not depend on (past the end the first item of all, not used)
  uint32_t k;
  int v;
  auto load = [&](int i) {
    const int ic = i < end ? i : 0;
    k = kin[ic];
    v = vin ? vin[ic] : ic;
  };
  load(blk * span + threadIdx.x);
  digit_positions(hist, blk, nb, span, pos, reinterpret_cast<int*>(wcnt), wsum);
  __syncthreads();
  for (int d = threadIdx.x; d < kSortDigits; d += kSortThreads) wcnt[d] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  for (int i0 = blk * span; i0 < end; i0 += kSortThreads) {
    const bool valid = i0 + (int)threadIdx.x < end;
    const uint32_t kk = k;
    const int vv = v;
    float x, y;
    if (kLast) {
      x = px[vv];
      y = py[vv];
    }
    load(i0 + kSortThreads + threadIdx.x);  // the next round's
    const int r = rank_items(key_digit(kk, pass), valid, i0 + kSortThreads < end, pos, wcnt);
    if (!valid) continue;
    vout[r] = vv;
    if (kLast) {
      irank[vv] = r;
      xs[r] = x;
      ys[r] = y;
    } else {
      kout[r] = kk;
    }
  }
}

template <bool kLast>
__global__ __launch_bounds__(kSortThreads) void sort_scatter_kernel(int n, int span, int pass,
                                                                    const uint32_t* __restrict__ kin,
                                                                    const int* __restrict__ vin,
                                                                    const SortCount* __restrict__ hist,
                                                                    uint32_t* __restrict__ kout,
                                                                    int* __restrict__ vout,
                                                                    const float* __restrict__ px,
                                                                    const float* __restrict__ py,
                                                                    int* __restrict__ irank, float* __restrict__ xs,
                                                                    float* __restrict__ ys) {
  __shared__ ScatterLds lds;
  sort_scatter_body<kLast>(lds, gridDim.x, n, span, pass, kin, vin, hist, kout, vout, px, py, irank, xs, ys);
}

template <bool kScaled>
__global__ __launch_bounds__(256) void plan_tiles_kernel(int n, int nrt, float s2, int* perm, float* __restrict__ xs,
                                                         float* __restrict__ ys, float4* cbox, float4* sbox,
                                                         float* __restrict__ xc, float* __restrict__ yc,
                                                         float2* __restrict__ cen) {
  plan_tiles_block<kScaled>(blockIdx.x, n, nrt, s2, perm, xs, ys, cbox, sbox, xc, yc, cen);
}

// ---- lists of live chunks ----

// Subtile masks of one (row tile, chunk) pair: bit t when subtile t sees the
// chunk, bit 4 + t when that pair also needs the lo part; 0 when none does.
__device__ __forceinline__ unsigned pair_mask(const float4 (&sb)[kSubsPerTile], const float4& rb, const float4& q,
                                              float s2, float threshold, float lo_threshold) {
  unsigned mask = 0u;
  if (boxes_live(rb, q, s2, threshold)) {
#pragma unroll
    for (int t = 0; t < kSubsPerTile; ++t) {
      mask |= (boxes_live(sb[t], q, s2, threshold) ? 1u : 0u) << t;
      mask |= (boxes_live(sb[t], q, s2, lo_threshold) ? 1u : 0u) << (4 + t);
    }
  }
  return (mask & 0xfu) != 0u ? mask : 0u;
}
__device__ __forceinline__ float4 row_box(const float4* cbox, int r) {
  float4 rb = cbox[kChunksPerTile * r];
#pragma unroll
  for (int t = 1; t < kChunksPerTile; ++t) rb = join_extent(rb, cbox[kChunksPerTile * r + t]);
  return rb;
}

// One workgroup of four waves per row tile: the ascending list of its live
// chunks, 1024 chunks a round (four box loads of a lane in flight), compacted by
// ballots; the row tile's cost.
constexpr int kListBatch = 4;
__device__ __forceinline__ void row_list(int r, int nch, const float4* __restrict__ cbox,
                                         const float4* __restrict__ sbox, float s2, float threshold,
                                         float lo_threshold, int* count, uint32_t* list, int* roww) {
  __shared__ int cnt_s[4 * kListBatch];
  __shared__ int cost_s[4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  float4 sb[kSubsPerTile];
#pragma unroll
  for (int t = 0; t < kSubsPerTile; ++t) sb[t] = sbox[kSubsPerTile * r + t];
  const float4 rb = row_box(cbox, r);
  uint32_t* out = list + (size_t)r * nch;
  int base = 0, cost = 0;
  for (int c0 = 0; c0 < nch; c0 += 4 * kListBatch * 64) {
    float4 q[kListBatch];
    unsigned mask[kListBatch];
    unsigned long long bal[kListBatch];
#pragma unroll
    for (int u = 0; u < kListBatch; ++u) q[u] = cbox[min(c0 + (wv * kListBatch + u) * 64 + lane, nch - 1)];
#pragma unroll
    for (int u = 0; u < kListBatch; ++u) {
      const int c = c0 + (wv * kListBatch + u) * 64 + lane;
      mask[u] = c < nch ? pair_mask(sb, rb, q[u], s2, threshold, lo_threshold) : 0u;
      bal[u] = __ballot(mask[u] != 0u);
      if (lane == 0) cnt_s[wv * kListBatch + u] = __popcll(bal[u]);
    }
    __syncthreads();
    int before[kListBatch];
#pragma unroll
    for (int b = 0; b < 4 * kListBatch; ++b) {
#pragma unroll
      for (int u = 0; u < kListBatch; ++u)
        if (b == wv * kListBatch + u) before[u] = base;
      base += cnt_s[b];
    }
#pragma unroll
    for (int u = 0; u < kListBatch; ++u)
      if (mask[u]) {
        const uint32_t e = (uint32_t)(c0 + (wv * kListBatch + u) * 64 + lane) | (mask[u] << 16);
        out[before[u] + __popcll(bal[u] & ((1ull << lane) - 1ull))] = e;
        cost += unit_cost(e);
      }
    __syncthreads();  // cnt_s is rewritten by the next round
  }
  cost = warp_sum(cost);
  if (lane == 0) cost_s[wv] = cost;
  __syncthreads();
  if (threadIdx.x == 0) {
    count[r] = base;
    roww[r] = kCostRowTile + cost_s[0] + cost_s[1] + cost_s[2] + cost_s[3];
  }
}

__global__ __launch_bounds__(256) void plan_lists_kernel(int nch, const float4* __restrict__ cbox,
                                                         const float4* __restrict__ sbox, float s2, float threshold,
                                                         float lo_threshold, int* count, uint32_t* list, int* roww) {
  row_list(blockIdx.x, nch, cbox, sbox, s2, threshold, lo_threshold, count, list, roww);
}

// And by the workgroups after the row tiles' the column maxima of right-hand sides
// that were formed beside the boxes, too late for plan_extent_rhs_kernel.
__global__ __launch_bounds__(256) void plan_lists_rhs_kernel(int nrt, int nch, const float4* __restrict__ cbox,
                                                             const float4* __restrict__ sbox, float s2,
                                                             float threshold, float lo_threshold, int* count,
                                                             uint32_t* list, int* roww, RhsJob J) {
  __shared__ float red[4];
  if ((int)blockIdx.x < nrt) row_list(blockIdx.x, nch, cbox, sbox, s2, threshold, lo_threshold, count, list, roww);
  else colmax_unit(J, blockIdx.x - nrt, threadIdx.x, red);
}

// Exclusive prefix sum of n ints in one workgroup of 1024 threads (in place
// allowed); the sum goes to *sum. A round covers 16384 entries: they are loaded
// into LDS with coalesced loads, each thread scans 16 consecutive ones (row
// stride 17 words, so the 64 lanes of a wave hit distinct banks), the thread
// totals are scanned across the workgroup, and the results go back through LDS
// to coalesced stores. T (the output type) is int or long long.
constexpr int kScanIpt = 16;
constexpr int kScanRound = 1024 * kScanIpt;
template <class T>
__global__ __launch_bounds__(1024) void plan_scan_kernel(int n, const int* in, T* out, T* sum) {
  __shared__ T buf[1024 * (kScanIpt + 1)];
  __shared__ T wsum[16];
  __shared__ T carry_s;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (tid == 0) carry_s = 0;
  for (int base = 0; base < n; base += kScanRound) {
    __syncthreads();  // the previous round's stores have read buf
#pragma unroll
    for (int k = 0; k < kScanIpt; ++k) {
      const int e = k * 1024 + tid;  // entry of the round, coalesced
      buf[(e / kScanIpt) * (kScanIpt + 1) + e % kScanIpt] = base + e < n ? (T)in[base + e] : (T)0;
    }
    __syncthreads();
    T* row = buf + tid * (kScanIpt + 1);
    T tot = 0;
#pragma unroll
    for (int k = 0; k < kScanIpt; ++k) tot += row[k];
    T x = tot;  // inclusive scan of the thread totals within the wave
    for (int off = 1; off < 64; off <<= 1) {
      const T y = __shfl_up(x, off, 64);
      if (lane >= off) x += y;
    }
    if (lane == 63) wsum[wv] = x;
    __syncthreads();
    T before = carry_s;
    for (int k = 0; k < wv; ++k) before += wsum[k];
    T run = before + x - tot;
#pragma unroll
    for (int k = 0; k < kScanIpt; ++k) {
      const T v = row[k];
      row[k] = run;
      run += v;
    }
    __syncthreads();
    if (tid == 1023) carry_s = before + x;
#pragma unroll
    for (int k = 0; k < kScanIpt; ++k) {
      const int e = k * 1024 + tid;
      if (base + e < n) out[base + e] = buf[(e / kScanIpt) * (kScanIpt + 1) + e % kScanIpt];
    }
  }
  __syncthreads();
  if (tid == 0) *sum = carry_s;
}

// Largest row tile r with unit_off[r] <= u.
__device__ __forceinline__ int row_of_unit(const int* unit_off, int nrt, int u) {
  int lo = 0, hi = nrt - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (unit_off[mid] <= u) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Largest wave w with wunit[w] <= u (the wave whose range holds unit u).
__device__ __forceinline__ int wave_of_unit(int u, const int* wunit, int nw) {
  int lo = 0, hi = nw - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (wunit[mid] <= u) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Units of a row tile's list L (cnt of them) whose cost before them, the row
// tile's own included, is below rem: by one wave, 64 units at a time, the loads of
// four such groups in flight together (a wave that waited for each group on its own
// spent most of its time there).
__device__ __forceinline__ int units_before(const uint32_t* L, int cnt, long long rem, int lane) {
  constexpr int kGroups = 4;
  long long before = kCostRowTile;  // cost up to the current group of 64 units
  int k = 0;
  for (int k0 = 0; k0 < cnt && before < rem; k0 += 64 * kGroups) {
    uint32_t e[kGroups];
#pragma unroll
    for (int g = 0; g < kGroups; ++g) e[g] = L[min(k0 + 64 * g + lane, cnt - 1)];
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      if (k0 + 64 * g >= cnt) break;
      const int kk = k0 + 64 * g + lane;
      const int c = kk < cnt ? unit_cost(e[g]) : 0;
      const int x = warp_prefix(c);  // within the group
      k += __popcll(__ballot(kk < cnt && before + (x - c) < rem));
      before += __builtin_amdgcn_readlane(x, 63);
    }
  }
  return k;
}

// First unit of each wave b in [0, nw]: the first unit whose exclusive cost
// prefix reaches the wave's target, wtot x (round weight of the waves below b)
// / (that of all nw waves). A row tile's own cost counts before its first unit.
// One wave per boundary: the row tile by binary search over the row prefixes,
// then the units of that row tile 64 at a time.
__global__ __launch_bounds__(256) void plan_wunit_kernel(int nrt, int nch, int nw, int wround, const int* count,
                                                         const uint32_t* __restrict__ list, const int* unit_off,
                                                         const long long* rowwoff, const long long* wtot, int* wunit) {
  const int b = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (b > nw) return;
  const long long t = *wtot * wave_weight_below(b, wround) / wave_weight_below(nw, wround);
  int lo = 0, hi = nrt - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (rowwoff[mid] <= t) lo = mid; else hi = mid - 1;
  }
  const int r = lo;
  const int k = units_before(list + (size_t)r * nch, count[r], t - rowwoff[r], lane);
  if (lane == 0) wunit[b] = unit_off[r] + k;
}

// Per wave: first row tile and number of row tiles its units touch (the count
// goes to nrows[w], scanned into partial slots afterwards).
__global__ void plan_waves_kernel(int nrt, int nw, const int* wunit, const int* unit_off, int* wrow, int* nrows) {
  const int w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= nw) return;
  const int u0 = wunit[w], u1 = wunit[w + 1];
  if (u0 >= u1) {
    wrow[w] = -1;
    nrows[w] = 0;
    return;
  }
  const int r0 = row_of_unit(unit_off, nrt, u0), r1 = row_of_unit(unit_off, nrt, u1 - 1);
  wrow[w] = r0;
  nrows[w] = r1 - r0 + 1;
}

// Per row tile: its partial slots [s0, s0 + cnt), from the first and last wave
// holding its units (waves in between start in this row tile, so their slots
// for it are their first ones, and empty waves own no slot).
__global__ void plan_rowslots_kernel(int nrt, int nw, const int* wunit, const int* unit_off, const int* count,
                                     const int* wrow, const int* wslot, int2* rslot) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nrt) return;
  const int a = unit_off[r], c = count[r];
  if (c <= 0) {
    rslot[r] = make_int2(0, 0);
    return;
  }
  const int wf = wave_of_unit(a, wunit, nw), wl = wave_of_unit(a + c - 1, wunit, nw);
  const int s0 = wslot[wf] + (r - wrow[wf]);
  const int s1 = wslot[wl] + (r - wrow[wl]);
  rslot[r] = make_int2(s0, s1 - s0 + 1);
}

// Per wave, its range in one load: the first row tile r, its first partial
// slot, the list positions [kb, ke) it takes in row tile r, and the number of
// units it takes in the row tiles after r (-1 row tile: no units).
__global__ void plan_wdesc_kernel(int nw, const int* wunit, const int* unit_off, const int* count, const int* wrow,
                                  const int* wslot, int4* wdesc, int* wrest) {
  const int w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= nw) return;
  const int u0 = wunit[w], u1 = wunit[w + 1];
  const int r = wrow[w];
  if (u0 >= u1 || r < 0) {
    wdesc[w] = make_int4(-1, wslot[w], 0, 0);
    wrest[w] = 0;
    return;
  }
  const int off = unit_off[r];
  const int ke = min(u1, off + count[r]) - off;
  wdesc[w] = make_int4(r, wslot[w], u0 - off, ke);
  wrest[w] = u1 - (off + ke);
}

// ---- the same split with fewer launches, for up to kFoldRows row tiles ----

constexpr int kFoldRows = 4096;

// Exclusive prefixes of the row tiles' unit counts and costs, off and woff (LDS,
// nrt <= kFoldRows), by a workgroup of NT threads; returns the total cost.
static_assert(kFoldRows * (kCostRowTile + (long long)kChunksPerTile * kFoldRows * kMostUnitCost) < 1ll << 31,
              "32-bit costs");
template <int NT>
__device__ __forceinline__ int fold_rows(int nrt, const int* __restrict__ count, const int* __restrict__ roww,
                                         int* off, int* woff) {
  __shared__ int cs[NT / 64], ws[NT / 64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  for (int r = tid; r < nrt; r += NT) {
    off[r] = count[r];
    woff[r] = roww[r];
  }
  __syncthreads();
  const int per = cdiv(nrt, NT), r0 = min(tid * per, nrt), r1 = min(r0 + per, nrt);
  int c = 0, v = 0;
  for (int r = r0; r < r1; ++r) {
    c += off[r];
    v += woff[r];
  }
  int xc = warp_prefix(c), xv = warp_prefix(v);
  if (lane == 63) {
    cs[w] = xc;
    ws[w] = xv;
  }
  __syncthreads();
  xc -= c;
  xv -= v;
  int total = 0;
  for (int k = 0; k < NT / 64; ++k) {
    if (k < w) {
      xc += cs[k];
      xv += ws[k];
    }
    total += ws[k];
  }
  for (int r = r0; r < r1; ++r) {
    const int cr = off[r], vr = woff[r];
    off[r] = xc;
    woff[r] = xv;
    xc += cr;
    xv += vr;
  }
  __syncthreads();
  return total;
}

// Largest index k in [0, n) with v[k] <= u (v ascending, v[0] <= u).
template <class T>
__device__ __forceinline__ int last_at_most(const T* v, int n, T u) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (v[mid] <= u) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// The same by one wave, all its lanes with the same arguments: 64 entries a look.
template <class T>
__device__ __forceinline__ int wave_last_at_most(const T* v, int n, T u, int lane) {
  int lo = 0, len = n;
  while (len > 1) {
    const int step = cdiv(len, 64), at = lane * step;
    const int j = __popcll(__ballot(at < len && v[lo + min(at, len - 1)] <= u)) - 1;
    lo += j * step;
    len = min(step, len - j * step);
  }
  return lo;
}

// The row tiles of the units on both sides of a boundary at unit u: (of u - 1, of u).
__device__ __forceinline__ int2 boundary_rows(const int* off, int nrt, int u) {
  const int r = last_at_most(off, nrt, u);
  return make_int2(u > 0 && off[r] == u ? last_at_most(off, nrt, u - 1) : r, r);
}

// plan_wunit_kernel with the prefixes of the row tiles formed by every workgroup
// itself; the first one writes unit_off. Bound by latency, so few row tiles are left
// to a thread (512 threads past kFewRows row tiles; below, the larger workgroups take
// longer to start: 5.8 us instead of 5.3 at 88 row tiles), and the searches look at 64
// entries at a time. 4.5 us at 88 row tiles, 7.6 at 625 and 8.6 at 2500, where 256
// threads, binary searches and lists read 64 units at a time took 5.0, 9.6 and 14.1;
// with the prefixes by DPP 6.5 at 625.
constexpr int kFewRows = 256;
template <int NT>
__global__ __launch_bounds__(NT) void plan_wunit_fold_kernel(int nrt, int nch, int nw, int wround, const int* count,
                                                             const uint32_t* __restrict__ list, const int* roww,
                                                             int* unit_off, int* wunit, int2* wrows) {
  __shared__ int off[kFoldRows];
  __shared__ int woff[kFoldRows];
  const long long wtot = fold_rows<NT>(nrt, count, roww, off, woff);
  if (blockIdx.x == 0)
    for (int r = threadIdx.x; r < nrt; r += NT) unit_off[r] = off[r];
  const int b = blockIdx.x * (NT / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (b > nw) return;
  const int t = (int)(wtot * wave_weight_below(b, wround) / wave_weight_below(nw, wround));
  const int r = wave_last_at_most(woff, nrt, t, lane), cnt = count[r];
  const int u = off[r] + units_before(list + (size_t)r * nch, cnt, t - woff[r], lane);
  const int ru = wave_last_at_most(off, nrt, u, lane);
  const int rb = u > 0 && off[ru] == u ? wave_last_at_most(off, nrt, u - 1, lane) : ru;
  if (lane == 0) {
    wunit[b] = u;
    wrows[b] = make_int2(rb, ru);
  }
}

// Ranges and partial slots of all waves, and the slots of every row tile, by one
// workgroup of 1024 threads. off: first unit of each row tile; wunit, wrows: the
// units and row tiles at the nw + 1 boundaries; wslot: scratch (LDS). A wave knows
// where its row tiles' units start and end, so it writes the ends of their ranges
// of slots itself (first, and one past the last, in LDS; a slot index is below
// kMaxPlanWaves + kFoldRows); empty row tiles keep an empty range.
static_assert(kMaxPlanWaves + kFoldRows < 65536 && kChunksPerTile * kFoldRows < 65536, "16-bit slots and counts");
template <class Count>
__device__ __forceinline__ void finish_waves(int nrt, int nw, const int* off, const Count* count, const int* wunit,
                                             const int2* wrows, int* wslot, unsigned short* first,
                                             unsigned short* past, int2* __restrict__ rslot,
                                             int4* __restrict__ wdesc, int* __restrict__ wrest) {
  __shared__ int ws[1024 / 64];
  const int tid = threadIdx.x;
  for (int r = tid; r < nrt; r += 1024) {
    first[r] = 0;
    past[r] = 0;
  }
  const int per = cdiv(nw, 1024), w0 = min(tid * per, nw), w1 = min(w0 + per, nw);
  int sum = 0;
  for (int w = w0; w < w1; ++w) {
    const int rows = wunit[w] < wunit[w + 1] ? wrows[w + 1].x - wrows[w].y + 1 : 0;
    wslot[w] = rows;
    sum += rows;
  }
  int run = block_exclusive(sum, ws);
  for (int w = w0; w < w1; ++w) {
    const int rows = wslot[w];
    wslot[w] = run;
    run += rows;
  }
  __syncthreads();
  for (int w = tid; w < nw; w += 1024) {
    const int u0 = wunit[w], u1 = wunit[w + 1], slot = wslot[w];
    int4 dsc = make_int4(-1, slot, 0, 0);
    int rest = 0;
    if (u0 < u1) {
      const int r0 = wrows[w].y, r1 = wrows[w + 1].x;
      for (int r = r0; r <= r1; ++r) {
        const int c = count[r];
        if (c <= 0) continue;  // its (unused) slot stays with the wave
        if (u0 <= off[r]) first[r] = (unsigned short)(slot + (r - r0));
        if (u1 >= off[r] + c) past[r] = (unsigned short)(slot + (r - r0) + 1);
      }
      const int o = off[r0], ke = min(u1, o + count[r0]) - o;
      dsc = make_int4(r0, slot, u0 - o, ke);
      rest = u1 - (o + ke);
    }
    wdesc[w] = dsc;
    wrest[w] = rest;
  }
  __syncthreads();
  for (int r = tid; r < nrt; r += 1024) rslot[r] = make_int2(first[r], past[r] - first[r]);
}

__device__ __forceinline__ void plan_finish_body(int nrt, int nw, const int* __restrict__ unit_off,
                                                 const int* __restrict__ count_g, const int* __restrict__ wunit,
                                                 const int2* __restrict__ wrows, int2* __restrict__ rslot,
                                                 int4* __restrict__ wdesc, int* __restrict__ wrest) {
  __shared__ int off[kFoldRows], wslot[kMaxPlanWaves];
  __shared__ unsigned short count[kFoldRows], first[kFoldRows], past[kFoldRows];
  for (int r = threadIdx.x; r < nrt; r += 1024) {
    off[r] = unit_off[r];
    count[r] = (unsigned short)count_g[r];
  }
  finish_waves(nrt, nw, off, count, wunit, wrows, wslot, first, past, rslot, wdesc, wrest);
}

__global__ __launch_bounds__(1024) void plan_finish_kernel(int nrt, int nw, const int* __restrict__ unit_off,
                                                           const int* __restrict__ count,
                                                           const int* __restrict__ wunit,
                                                           const int2* __restrict__ wrows, int2* __restrict__ rslot,
                                                           int4* __restrict__ wdesc, int* __restrict__ wrest) {
  plan_finish_body(nrt, nw, unit_off, count, wunit, wrows, rslot, wdesc, wrest);
}

// And the right-hand sides by the workgroups after the first.
__global__ __launch_bounds__(1024) void plan_finish_rhs_kernel(int nrt, int nw, const int* __restrict__ unit_off,
                                                               const int* __restrict__ count,
                                                               const int* __restrict__ wunit,
                                                               const int2* __restrict__ wrows,
                                                               int2* __restrict__ rslot, int4* __restrict__ wdesc,
                                                               int* __restrict__ wrest, RhsJob J) {
  __shared__ int se[1024 / 256][kPlaceSlots];
  if (blockIdx.x == 0) {
    plan_finish_body(nrt, nw, unit_off, count, wunit, wrows, rslot, wdesc, wrest);
  } else {
    // past what the L2s hold (40 MB at 160,000 points and 64 columns) an XCD takes
    // neighbouring points: their rows of V share cache lines
    const int g = threadIdx.x >> 8, per = round_up(cdiv(J.b.ldh, 1024), kXcds), u = blockIdx.x - 1;
    const int bx = per > 64 ? xcd_block(u % per, per) : u % per;
    place_unit(J, bx * (1024 / 256) + g, u / per * kPlaceSlots, threadIdx.x & 255, se[g]);
  }
}

// ---- small point sets: the whole plan by one workgroup ----

// Up to kSmallPoints points a launch costs more than its work: one workgroup of
// 1024 threads keeps the keys, the order and the split in LDS and writes the plan
// (or, without kPlan, the sorted points and boxes).
constexpr int kSmallPoints = 4096;
constexpr int kSmallTiles = kSmallPoints / kRowTile, kSmallChunks = kSmallTiles * kChunksPerTile;
static_assert(kSortThreads == 1024, "one workgroup size for the sort and the small plan");

constexpr int kSmallRounds = kSmallPoints / kSortThreads;  // items a thread
constexpr int kSmallBits = 6, kSmallPasses = 2 * kHilbertBits / kSmallBits;
static_assert(1 << kSmallBits == 64 && kSmallPasses * kSmallBits == 2 * kHilbertBits, "a lane per digit");

union SmallLds {
  ScatterLds rank;  // of the large set sorted beside (sort_scatter_side_kernel)
  struct {
    uint32_t key[2][kSmallPoints];
    int cnt[64 * (kSmallRounds * kSortThreads / 64 + 1)];
  } sort;
  struct {
    unsigned short cost[kSmallTiles][kSmallChunks];  // cost of a row tile before each of its units
    int wunit[8 * kSmallTiles + 1], wslot[8 * kSmallTiles];
    int2 wrows[8 * kSmallTiles + 1];
    int off[kSmallTiles], count[kSmallTiles], roww[kSmallTiles];
    unsigned short first[kSmallTiles], past[kSmallTiles];
    int woff[kSmallTiles];
    float4 cbox[kSmallChunks], sbox[kSmallTiles * kSubsPerTile];
  } plan;
};

// Stable order of the keys in L.sort.key[0], six bits a pass. A group of 64 items (wave
// w in round k) counts its digits in a column of cnt, lane by lane; the prefix of cnt
// along the digits, the groups of each in turn, gives every group's first position of a
// digit. Bound by the issue of one compute unit: two sets of 4,096 and 576 points take
// 26.4 us (28.9 with 12 bits a pass, 80 KB of counters cleared for each and the rounds
// ranked in turn). The whole plan of 576 points takes 14.2 us, 16.0 before the prefixes
// were taken by DPP.
__device__ __forceinline__ const unsigned short* small_order(SmallLds& L, int n,
                                                             unsigned short (&val)[2][kSmallPoints], int* ws) {
  constexpr int kWaves = kSortThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int R = cdiv(n, kSortThreads), row = R * kWaves + 1;  // one more: lanes fall on distinct banks
  int* const cnt = L.sort.cnt;
  for (int pass = 0; pass < kSmallPasses; ++pass) {
    const uint32_t* kin = L.sort.key[pass & 1];
    const unsigned short* vin = val[~pass & 1];
    uint32_t key[kSmallRounds];
    int v[kSmallRounds], at[kSmallRounds], lower[kSmallRounds];
#pragma unroll
    for (int k = 0; k < kSmallRounds; ++k) {
      if (k >= R) break;
      const int i = k * kSortThreads + tid, g = k * kWaves + w;
      const bool valid = i < n;
      cnt[lane * row + g] = 0;
      if (k * kSortThreads + w * 64 >= n) continue;  // no item in the group
      __builtin_amdgcn_wave_barrier();  // a wave's own LDS stores stay in order
      key[k] = valid ? kin[i] : 0u;
      v[k] = valid && pass > 0 ? (int)vin[i] : i;
      const int d = (int)(key[k] >> (kSmallBits * pass)) & 63;
      unsigned long long m = __ballot(valid);
#pragma unroll
      for (int b = 0; b < kSmallBits; ++b) {
        const bool bit = (d >> b) & 1;
        const unsigned long long bb = __ballot(bit);
        m &= bit ? bb : ~bb;
      }
      lower[k] = __popcll(m & ((1ull << lane) - 1ull));
      at[k] = d * row + g;
      if (valid && lower[k] == 0) cnt[at[k]] = __popcll(m);
    }
    __syncthreads();
    int* const mine = cnt + (tid / kWaves) * row + tid % kWaves * R;  // R entries of digit tid / kWaves
    int c[kSmallRounds], sum = 0;
#pragma unroll
    for (int k = 0; k < kSmallRounds; ++k) {
      c[k] = k < R ? mine[k] : 0;
      sum += c[k];
    }
    int run = block_exclusive(sum, ws);
#pragma unroll
    for (int k = 0; k < kSmallRounds; ++k) {
      if (k >= R) break;
      mine[k] = run;
      run += c[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSmallRounds; ++k) {
      if (k >= R || k * kSortThreads + tid >= n) break;
      const int r = cnt[at[k]] + lower[k];
      L.sort.key[~pass & 1][r] = key[k];
      val[pass & 1][r] = (unsigned short)v[k];
    }
    __syncthreads();
  }
  return val[(kSmallPasses - 1) & 1];
}

template <bool kPlan>
__device__ __forceinline__ void plan_small_body(SmallLds& L, int n, const float* __restrict__ px,
                                                const float* __restrict__ py, const TilePlan& P, int* perm, int* irank,
                                                float s2, float threshold, float lo_threshold) {
  __shared__ unsigned short val[2][kSmallPoints];
  __shared__ float4 red[kSortThreads / 64];
  __shared__ int ws[kSortThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  constexpr int kWaves = kSortThreads / 64;
  {
    const float4 e = wave_extent(thread_extent(n, px, py, tid, kSortThreads));
    if (lane == 0) red[w] = e;
    __syncthreads();
  }
  float4 ext = red[0];
  for (int k = 1; k < kWaves; ++k) ext = join_extent(ext, red[k]);
  ext = extent_square(ext);
  for (int i = tid; i < n; i += kSortThreads) L.sort.key[0][i] = point_key(px[i], py[i], ext);
  const unsigned short* order = small_order(L, n, val, ws);
  for (int tile = w; tile < P.nrt; tile += kWaves) {
    const int r = tile * kRowTile + lane;
    const bool live = r < n;
    const int v = live ? (int)order[r] : -1;
    const float x = live ? px[v] : 0.f, y = live ? py[v] : 0.f;
    perm[r] = v;
    if (live) irank[v] = r;
    P.xs[r] = x;
    P.ys[r] = y;
    tile_boxes<kPlan>(tile, x, y, live, s2, L.plan.cbox, L.plan.sbox, P.xc, P.yc, P.cen);  // the keys are done with
  }
  __syncthreads();
  for (int c = tid; c < P.nch; c += kSortThreads) P.cbox[c] = L.plan.cbox[c];
  for (int t = tid; t < P.nrt * kSubsPerTile; t += kSortThreads) P.sbox[t] = L.plan.sbox[t];
  if (!kPlan) return;
  for (int r = w; r < P.nrt; r += kWaves) {
    float4 sb[kSubsPerTile];
#pragma unroll
    for (int t = 0; t < kSubsPerTile; ++t) sb[t] = L.plan.sbox[kSubsPerTile * r + t];
    const float4 rb = row_box(L.plan.cbox, r);
    uint32_t* out = P.list + (size_t)r * P.nch;
    int base = 0, before = kCostRowTile;  // units so far, and the row tile's cost up to them
    for (int c0 = 0; c0 < P.nch; c0 += 64) {
      const int c = c0 + lane;
      const unsigned mask = c < P.nch ? pair_mask(sb, rb, L.plan.cbox[c], s2, threshold, lo_threshold) : 0u;
      const unsigned long long bal = __ballot(mask != 0u);
      const uint32_t e = (uint32_t)c | (mask << 16);
      const int cost = mask ? unit_cost(e) : 0;
      const int x = warp_prefix(cost);
      if (mask) {
        const int k = base + __popcll(bal & ((1ull << lane) - 1ull));
        out[k] = e;
        L.plan.cost[r][k] = (unsigned short)(before + x - cost);
      }
      base += __popcll(bal);
      before += __builtin_amdgcn_readlane(x, 63);
    }
    if (lane == 0) {
      P.count[r] = L.plan.count[r] = base;
      L.plan.roww[r] = before;
    }
  }
  __syncthreads();
  const int nrt = P.nrt, nw = P.nw;
  // prefixes of the row tiles' unit counts and costs, a lane per row tile
  static_assert(kSmallTiles <= 64, "a wave holds the row tiles");
  int wtot;
  {
    const int c = lane < nrt ? L.plan.count[lane] : 0, v = lane < nrt ? L.plan.roww[lane] : 0;
    const int xc = warp_prefix(c), xv = warp_prefix(v);
    wtot = __builtin_amdgcn_readlane(xv, 63);
    if (w == 0 && lane < nrt) {
      L.plan.off[lane] = xc - c;
      L.plan.woff[lane] = xv - v;
    }
  }
  __syncthreads();
  // cost and weight fit 32 bits, and so does their product
  constexpr long long kMostCost = kSmallTiles * (kCostRowTile + (long long)kSmallChunks * kMostUnitCost);
  static_assert(kMostCost * 8 * kSmallTiles * kRoundWeight[0] < 1ll << 32, "32-bit targets");
  const unsigned wall = (unsigned)wave_weight_below(nw, P.wround);
  for (int b = tid; b <= nw; b += kSortThreads) {
    const int t = (int)((unsigned)wtot * (unsigned)wave_weight_below(b, P.wround) / wall);
    const int r = last_at_most(L.plan.woff, nrt, t);
    const int rem = t - L.plan.woff[r];
    int lo = 0, hi = L.plan.count[r];  // units whose cost before them is below rem
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if ((int)L.plan.cost[r][mid] < rem) lo = mid + 1; else hi = mid;
    }
    const int u = L.plan.off[r] + lo;
    L.plan.wunit[b] = u;
    L.plan.wrows[b] = boundary_rows(L.plan.off, nrt, u);
  }
  __syncthreads();
  finish_waves(nrt, nw, L.plan.off, L.plan.count, L.plan.wunit, L.plan.wrows, L.plan.wslot, L.plan.first, L.plan.past,
               P.rslot, P.wdesc, P.wrest);
}

template <bool kPlan>
__global__ __launch_bounds__(kSortThreads) void plan_small_kernel(int n, const float* __restrict__ px,
                                                                  const float* __restrict__ py, TilePlan P, int* perm,
                                                                  int* irank, float s2, float threshold,
                                                                  float lo_threshold) {
  __shared__ SmallLds lds;
  plan_small_body<kPlan>(lds, n, px, py, P, perm, irank, s2, threshold, lo_threshold);
}

// A small set to be sorted beside another one.
struct SmallSort {
  int n;
  const float *px, *py;
  TilePlan plan;
  int *perm, *irank;
};
static SmallSort small_sort(const TilePlan& p, int n, const float* px, const float* py) {
  return SmallSort{n, px, py, p, const_cast<int*>(p.perm), const_cast<int*>(p.irank)};
}
__device__ __forceinline__ void sort_small(SmallLds& lds, const SmallSort& s) {
  plan_small_body<false>(lds, s.n, s.px, s.py, s.plan, s.perm, s.irank, 1.f, 0.f, 0.f);
}

// Two small sets, a workgroup each.
__global__ __launch_bounds__(kSortThreads) void sort_small_pair_kernel(SmallSort a, SmallSort b) {
  __shared__ SmallLds lds;
  if (blockIdx.x == 0) sort_small(lds, a);
  else sort_small(lds, b);
}

// The first scatter pass of a large set, and a small set by a workgroup more: on its
// own that workgroup takes as long as the pass (some 17 us for 1600 points).
__global__ __launch_bounds__(kSortThreads) void sort_scatter_side_kernel(int n, int span, const uint32_t* kin,
                                                                         const SortCount* hist, uint32_t* kout,
                                                                         int* vout, SmallSort side) {
  __shared__ SmallLds lds;
  if (blockIdx.x + 1 == gridDim.x) sort_small(lds, side);
  else sort_scatter_body<false>(lds.rank, gridDim.x - 1, n, span, 0, kin, nullptr, hist, kout, vout, nullptr, nullptr,
                                nullptr, nullptr, nullptr);
}

// Compute units of the current device (queried once per device).
static int compute_units() {
  static int cached[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] <= 0) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
    cached[dev] = v;
  }
  return cached[dev];
}

// Sort of more than kSmallPoints points, and (kScaled) the scaled coordinates;
// pair (nullable): a small set sorted in the same launches; job (nullable): the column
// maxima of its right-hand sides too; side (nullable): work without need of the order.
template <bool kScaled>
static int sort_points(TilePlan& p, int n, const float* px, const float* py, float s2, const SmallSort* pair,
                       const RhsJob* job, const PlanSide* side, hipStream_t stream) {
  int* perm = const_cast<int*>(p.perm);
  int* irank = const_cast<int*>(p.irank);
  const int span = sort_span(n), nb = cdiv(n, span);
  // sort scratch in buffers that are written only after the sort: the partial
  // extents in cbox, the keys in xc and yc
  float4* ext = p.cbox;
  uint32_t *k0 = reinterpret_cast<uint32_t*>(p.xc), *k1 = reinterpret_cast<uint32_t*>(p.yc);
  const int parts = nb < 64 ? nb : 64;  // of the extent, one per workgroup: a wave folds them
  if (job && job->f16)
    hipLaunchKernelGGL(plan_extent_rhs_kernel, dim3(parts + cdiv(job->nrhs * kColmaxBlocks, kSortThreads / 256)),
                       dim3(kSortThreads), 0, stream, n, px, py, parts, ext, *job);
  else
    hipLaunchKernelGGL(plan_extent_kernel, dim3(parts), dim3(kSortThreads), 0, stream, n, px, py, ext);
  GPL_LAUNCH_CHECK();
  hipLaunchKernelGGL(plan_keys_kernel, dim3(nb), dim3(kSortThreads), 0, stream, n, span, px, py, ext, parts, k0,
                     p.shist);
  GPL_LAUNCH_CHECK();
  static_assert(kSortPasses == 2, "a first and a last pass");
  if (pair)
    hipLaunchKernelGGL(sort_scatter_side_kernel, dim3(nb + 1), dim3(kSortThreads), 0, stream, n, span, k0, p.shist, k1,
                       p.sval, *pair);
  else
    hipLaunchKernelGGL(sort_scatter_kernel<false>, dim3(nb), dim3(kSortThreads), 0, stream, n, span, 0, k0, nullptr,
                       p.shist, k1, p.sval, px, py, irank, p.xs, p.ys);
  GPL_LAUNCH_CHECK();
  hipLaunchKernelGGL(sort_count_kernel, dim3(nb), dim3(kSortThreads), 0, stream, n, span, 1, k1, p.shist);
  GPL_LAUNCH_CHECK();
  hipLaunchKernelGGL(sort_scatter_kernel<true>, dim3(nb), dim3(kSortThreads), 0, stream, n, span, 1, k1, p.sval,
                     p.shist, nullptr, perm, px, py, irank, p.xs, p.ys);
  GPL_LAUNCH_CHECK();
  if (side) return plan_tiles_side_launch(p, n, s2, kScaled, *side, stream);
  hipLaunchKernelGGL(plan_tiles_kernel<kScaled>, dim3(cdiv(p.nrt, 4)), dim3(256), 0, stream, n, p.nrt, s2, perm, p.xs,
                     p.ys, p.cbox, p.sbox, p.xc, p.yc, p.cen);
  GPL_LAUNCH_CHECK();
  return GPL_OK;
}

template <bool kPlan>
static int small_plan(TilePlan& p, int n, const float* px, const float* py, float s2, float threshold,
                      float lo_threshold, hipStream_t stream) {
  hipLaunchKernelGGL(plan_small_kernel<kPlan>, dim3(1), dim3(kSortThreads), 0, stream, n, px, py, p,
                     const_cast<int*>(p.perm), const_cast<int*>(p.irank), s2, threshold, lo_threshold);
  GPL_LAUNCH_CHECK();
  return GPL_OK;
}

int plan_sort(TilePlan& p, int n, const float* px, const float* py, hipStream_t stream, const PlanSide* side) {
  GPL_REQUIRE(n >= 1, "plan needs at least one point");
  if (n > kSmallPoints) return sort_points<false>(p, n, px, py, 1.f, nullptr, nullptr, side, stream);
  if (side) GPL_TRY(plan_side_launch(*side, stream));
  return small_plan<false>(p, n, px, py, 1.f, 0.f, 0.f, stream);
}

int plan_sort_pair(TilePlan& a, int na, const float* ax, const float* ay, TilePlan& b, int nb, const float* bx,
                   const float* by, hipStream_t stream) {
  GPL_REQUIRE(na >= 1 && nb >= 1, "plan needs at least one point");
  if (nb > kSmallPoints) {
    GPL_TRY(plan_sort(a, na, ax, ay, stream));
    return plan_sort(b, nb, bx, by, stream);
  }
  const SmallSort side = small_sort(b, nb, bx, by);
  if (na > kSmallPoints) return sort_points<false>(a, na, ax, ay, 1.f, &side, nullptr, nullptr, stream);
  hipLaunchKernelGGL(sort_small_pair_kernel, dim3(2), dim3(kSortThreads), 0, stream, small_sort(a, na, ax, ay), side);
  GPL_LAUNCH_CHECK();
  return GPL_OK;
}

int plan_build(TilePlan& p, int n, const float* px, const float* py, const gpl_grid* grid, float s2, float threshold,
               float lo_threshold, hipStream_t stream, const RhsJob* job, bool* placed, const PlanSide* side) {
  if (placed) *placed = false;
  if (grid) {
    const int m = grid->n * grid->ss;
    GPL_REQUIRE(m > 0 && (long)m * m == n, "grid does not match n=%d", n);
  }
  GPL_REQUIRE(n >= 1, "plan needs at least one point");
  GPL_REQUIRE(p.nch <= kMaxPlanChunks, "n=%d exceeds the product's limit of %d points", n, kMaxPlanChunks * kChunk);
  p.wround = 4 * compute_units();
  if (n <= kSmallPoints) {
    if (side) GPL_TRY(plan_side_launch(*side, stream));
    return small_plan<true>(p, n, px, py, s2, threshold, lo_threshold, stream);
  }
  if (p.nrt > kFoldRows) job = nullptr;
  GPL_TRY(sort_points<true>(p, n, px, py, s2, nullptr, side ? nullptr : job, side, stream));
  if (side && job && job->f16)  // the columns are there since the launch before
    hipLaunchKernelGGL(plan_lists_rhs_kernel, dim3(p.nrt + job->nrhs * kColmaxBlocks), dim3(256), 0, stream, p.nrt,
                       p.nch, p.cbox, p.sbox, s2, threshold, lo_threshold, p.count, p.list, p.roww, *job);
  else
    hipLaunchKernelGGL(plan_lists_kernel, dim3(p.nrt), dim3(256), 0, stream, p.nch, p.cbox, p.sbox, s2, threshold,
                       lo_threshold, p.count, p.list, p.roww);
  GPL_LAUNCH_CHECK();
  if (p.nrt <= kFoldRows) {
    const auto split = [&](auto ntc) {
      constexpr int NT = decltype(ntc)::value;
      hipLaunchKernelGGL(plan_wunit_fold_kernel<NT>, dim3(cdiv(p.nw + 1, NT / 64)), dim3(NT), 0, stream, p.nrt, p.nch,
                         p.nw, p.wround, p.count, p.list, p.roww, p.unit_off, p.wunit,
                         reinterpret_cast<int2*>(p.wrow));
    };
    if (p.nrt <= kFewRows) split(std::integral_constant<int, 256>{}); else split(std::integral_constant<int, 512>{});
    GPL_LAUNCH_CHECK();
    if (job)
      hipLaunchKernelGGL(plan_finish_rhs_kernel,
                         dim3(1 + round_up(cdiv(job->b.ldh, 1024), kXcds) * (job->b.ncp / kPlaceSlots)), dim3(1024), 0,
                         stream, p.nrt, p.nw, p.unit_off, p.count, p.wunit, reinterpret_cast<int2*>(p.wrow), p.rslot,
                         p.wdesc, p.wrest, *job);
    else
      hipLaunchKernelGGL(plan_finish_kernel, dim3(1), dim3(1024), 0, stream, p.nrt, p.nw, p.unit_off, p.count, p.wunit,
                         reinterpret_cast<int2*>(p.wrow), p.rslot, p.wdesc, p.wrest);
    GPL_LAUNCH_CHECK();
    if (placed) *placed = job != nullptr;
    return GPL_OK;
  }
  hipLaunchKernelGGL(plan_scan_kernel<int>, dim3(1), dim3(1024), 0, stream, p.nrt, p.count, p.unit_off, p.total);
  GPL_LAUNCH_CHECK();
  hipLaunchKernelGGL(plan_scan_kernel<long long>, dim3(1), dim3(1024), 0, stream, p.nrt, p.roww, p.rowwoff, p.wtot);
  GPL_LAUNCH_CHECK();
  hipLaunchKernelGGL(plan_wunit_kernel, dim3(cdiv(p.nw + 1, 4)), dim3(256), 0, stream, p.nrt, p.nch, p.nw, p.wround,
                     p.count, p.list, p.unit_off, p.rowwoff, p.wtot, p.wunit);
  GPL_LAUNCH_CHECK();
  hipLaunchKernelGGL(plan_waves_kernel, dim3(cdiv(p.nw, 256)), dim3(256), 0, stream, p.nrt, p.nw, p.wunit,
                     p.unit_off, p.wrow, p.wslot);
  GPL_LAUNCH_CHECK();
  hipLaunchKernelGGL(plan_scan_kernel<int>, dim3(1), dim3(1024), 0, stream, p.nw, p.wslot, p.wslot, p.wslot + p.nw);
  GPL_LAUNCH_CHECK();
  hipLaunchKernelGGL(plan_rowslots_kernel, dim3(cdiv(p.nrt, 256)), dim3(256), 0, stream, p.nrt, p.nw, p.wunit,
                     p.unit_off, p.count, p.wrow, p.wslot, p.rslot);
  GPL_LAUNCH_CHECK();
  hipLaunchKernelGGL(plan_wdesc_kernel, dim3(cdiv(p.nw, 256)), dim3(256), 0, stream, p.nw, p.wunit, p.unit_off,
                     p.count, p.wrow, p.wslot, p.wdesc, p.wrest);
  GPL_LAUNCH_CHECK();
  return GPL_OK;
}

}  // namespace gpl
