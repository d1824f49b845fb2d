// Boxes and scaled coordinates of the tiles of a plan: by a launch of their own
// (tileplan.hip), or beside work that needs no sorted points (psf.hip).
#pragma once

#include <cmath>

#include "common.hpp"
#include "tileplan.hpp"

namespace gpl {

__device__ __forceinline__ float4 join_extent(const float4& a, const float4& b) {
  return make_float4(fminf(a.x, b.x), fmaxf(a.y, b.y), fminf(a.z, b.z), fmaxf(a.w, b.w));
}
// An extent joined with that of the lane whose index differs in bit OFF (lane_xor).
template <int OFF>
__device__ __forceinline__ float4 join_lane_xor(const float4& e) {
  auto other = [](float v) { return __builtin_bit_cast(float, lane_xor<OFF>(__builtin_bit_cast(unsigned, v))); };
  return join_extent(e, make_float4(other(e.x), other(e.y), other(e.z), other(e.w)));
}
constexpr float kInf = INFINITY;

// Boxes of one 64-point tile by a wave, lane = sorted point (x, y, live or
// padding): of every 16-point subtile and 32-point chunk, and (kScaled) the block
// centre and the scaled, block-centred coordinates (TilePlan::xc, yc, cen). A
// non-finite coordinate gives an infinite box (never dropped), no valid point an
// empty one (always dropped). The centre is the middle of the block's box, scaled
// and rounded to a multiple of 2^-12 (a float); xc = sqrt(s2) x - centre is formed
// in FP64 and rounded once.
template <bool kScaled>
__device__ __forceinline__ void tile_boxes(int tile, float x, float y, bool live, float s2, float4* cbox, float4* sbox,
                                           float* __restrict__ xc, float* __restrict__ yc, float2* __restrict__ cen) {
  const int lane = threadIdx.x & 63;
  const unsigned long long bad = __ballot(live && !(isfinite(x) && isfinite(y)));
  float4 e = live && isfinite(x) && isfinite(y) ? make_float4(x, x, y, y) : make_float4(kInf, -kInf, kInf, -kInf);
  static_assert(kSubTile == 16 && kChunk == 32 && kRowTile == 64, "steps of lane_xor");
  e = join_lane_xor<8>(e);
  e = join_lane_xor<4>(e);
  e = join_lane_xor<2>(e);
  e = join_lane_xor<1>(e);
  if ((bad >> (lane & ~(kSubTile - 1))) & ((1ull << kSubTile) - 1ull)) e = make_float4(-kInf, kInf, -kInf, kInf);
  if (lane % kSubTile == 0) sbox[tile * kSubsPerTile + lane / kSubTile] = e;
  e = join_lane_xor<16>(e);
  if (lane % kChunk == 0) cbox[tile * kChunksPerTile + lane / kChunk] = e;
  if (kScaled) {
    e = join_lane_xor<32>(e);
    const double sg = sqrt((double)s2);
    const double mx = 0.5 * ((double)e.x + (double)e.y), my = 0.5 * ((double)e.z + (double)e.w);
    const float cx = isfinite(mx) ? (float)(rint(mx * sg * 4096.0) / 4096.0) : 0.f;
    const float cy = isfinite(my) ? (float)(rint(my * sg * 4096.0) / 4096.0) : 0.f;
    const int r = tile * kRowTile + lane;
    xc[r] = (float)((double)(live ? x : 0.f) * sg - (double)cx);
    yc[r] = (float)((double)(live ? y : 0.f) * sg - (double)cy);
    if (lane == 0) cen[tile] = make_float2(cx, cy);
  }
}

// Those of four tiles by workgroup blk of 256 threads; the padding of the last tile.
template <bool kScaled>
__device__ __forceinline__ void plan_tiles_block(int blk, int n, int nrt, float s2, int* perm,
                                                 float* __restrict__ xs, float* __restrict__ ys, float4* cbox,
                                                 float4* sbox, float* __restrict__ xc, float* __restrict__ yc,
                                                 float2* __restrict__ cen) {
  const int tile = blk * 4 + (threadIdx.x >> 6);
  if (tile >= nrt) return;
  const int r = tile * kRowTile + (threadIdx.x & 63);
  const bool live = r < n;
  const float x = live ? xs[r] : 0.f, y = live ? ys[r] : 0.f;
  if (!live) {
    xs[r] = 0.f;
    ys[r] = 0.f;
    perm[r] = -1;
  }
  tile_boxes<kScaled>(tile, x, y, live, s2, cbox, sbox, xc, yc, cen);
}

}  // namespace gpl
