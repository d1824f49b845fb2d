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
  for (int off = kSubTile / 2; off > 0; off >>= 1) {
    e.x = fminf(e.x, __shfl_xor(e.x, off, 64));
    e.y = fmaxf(e.y, __shfl_xor(e.y, off, 64));
    e.z = fminf(e.z, __shfl_xor(e.z, off, 64));
    e.w = fmaxf(e.w, __shfl_xor(e.w, off, 64));
  }
  if ((bad >> (lane & ~(kSubTile - 1))) & ((1ull << kSubTile) - 1ull)) e = make_float4(-kInf, kInf, -kInf, kInf);
  if (lane % kSubTile == 0) sbox[tile * kSubsPerTile + lane / kSubTile] = e;
  static_assert(kChunk == 2 * kSubTile && kRowTile == 2 * kChunk, "pairs of boxes");
  auto pair = [](const float4& a, int off) {
    return join_extent(a, make_float4(__shfl_xor(a.x, off, 64), __shfl_xor(a.y, off, 64), __shfl_xor(a.z, off, 64),
                                      __shfl_xor(a.w, off, 64)));
  };
  e = pair(e, kSubTile);
  if (lane % kChunk == 0) cbox[tile * kChunksPerTile + lane / kChunk] = e;
  if (kScaled) {
    e = pair(e, kChunk);
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
