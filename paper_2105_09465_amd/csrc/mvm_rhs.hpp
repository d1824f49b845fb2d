// The right-hand-side block of a product in its buffers (mvm_mfma.hip): by launches of
// its own, or by workgroups beside the plan's (tileplan.hip).
#pragma once

#include "common.hpp"
#include "internal.hpp"
#include "tileplan.hpp"

namespace gpl {

constexpr float kKScale = 2048.f;  // 2^11 applied to the FP16 exp tile

// Columns V (caller order) of a product over the plan whose order is perm.
struct RhsJob {
  int n, nrhs, ldv;
  bool f16;  // precision form
  const float* V;
  const int* perm;
  ProdBufs b;
};

// Column-wise max |V| in two steps without atomics: kColmaxBlocks groups of 256
// threads per column write partial maxima (as bit patterns of non-negative
// floats), which the split folds. Unit u of nrhs kColmaxBlocks by threads t; red: 4
// floats of the group. The workgroup synchronises once.
__device__ __forceinline__ void colmax_unit(const RhsJob& J, int u, int t, float* red) {
  const int c = u / kColmaxBlocks, bx = u % kColmaxBlocks;
  float m = 0.f;
  if (c < J.nrhs) {
    const float* __restrict__ v = J.V + (size_t)c * J.ldv;
    constexpr int kU = 8, kStep = kColmaxBlocks * 256;
    for (int i0 = bx * 256 + t; i0 < J.n; i0 += kU * kStep) {
      float x[kU];  // loads issued together; past the end they repeat the first one
#pragma unroll
      for (int q = 0; q < kU; ++q) x[q] = v[i0 + q * kStep < J.n ? i0 + q * kStep : i0];
#pragma unroll
      for (int q = 0; q < kU; ++q) m = fmaxf(m, fabsf(x[q]));
    }
  }
  m = warp_max(m);
  if ((t & 63) == 0) red[t >> 6] = m;
  __syncthreads();
  if (t == 0 && c < J.nrhs) J.b.colmax[u] = __float_as_uint(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])));
}

// Sorted position j of column c: the caller's row perm[j] (or j), zero past n
// and for c >= nrhs.
__device__ __forceinline__ float gather_rhs(const RhsJob& J, int j, int c) {
  if (c >= J.nrhs || j >= J.n) return 0.f;
  return J.V[(size_t)c * J.ldv + (J.perm ? J.perm[j] : j)];
}

// Column of slot `slot` of the buffers: column `slot`, or in a packed last block
// (one FP16 part a slot, lo in odd ones) column b0 + (slot - b0) / 2.
__device__ __forceinline__ int slot_column(int slot, int nrhs, bool& packed) {
  const int b0 = packed_block_start(nrhs);
  packed = last_block_packed(nrhs) && slot >= b0;
  return packed ? b0 + (slot - b0) / 2 : slot;
}

// Exponent e of a column with the largest magnitude mx: mx 2^e in [2^13, 2^14); e
// is capped so that 2^e stays a finite float (a column below 2^-113 then scales
// to less than 2^13, still normal in FP16).
__device__ __forceinline__ int column_exponent(float mx) {
  return mx > 0.f && isfinite(mx) ? min(14 - ilogbf(mx) - 1, 126) : 0;
}

// V' = V * 2^e_c split into FP16 hi (nearest) and lo, in sorted order, position j
// of one slot; inv_scale[c] = 2^-e_c / 2^11 folds both scales for the output.
__device__ __forceinline__ void split_rhs_at(const RhsJob& J, int j, int slot, int c, bool packed, int e, float value) {
  const int b0 = packed_block_start(J.nrhs), ncp = J.b.ncp;
  _Float16 *Vh = J.b.Vh, *Vl = J.b.Vl;
  const float scale = ldexpf(1.f, e);
  if (j == 0 && c < ncp && (!packed || ((slot - b0) & 1) == 0)) J.b.inv_scale[c] = ldexpf(1.f, -e) / kKScale;
  const float v = value * scale;
  const _Float16 h = (_Float16)v;
  const _Float16 l = (_Float16)(v - (float)h);
  if (packed) {
    Vh[rhs_at(slot, j, ncp)] = ((slot - b0) & 1) ? l : h;
  } else {
    Vh[rhs_at(c, j, ncp)] = h;
    Vl[rhs_at(c, j, ncp)] = l;
  }
}

// kPlaceSlots slots by 256 threads t, a thread sorted position bx 256 + t of all of
// them: their gathers are in flight together. In the precision form wave w folds
// the partial maxima of slot w (se: kPlaceSlots ints of the group). The workgroup
// synchronises once.
constexpr int kPlaceSlots = 4;
static_assert(kColmaxBlocks <= 64, "a wave folds a column's partial maxima");
__device__ __forceinline__ void place_unit(const RhsJob& J, int bx, int slot0, int t, int* se) {
  const int j = bx * 256 + t, lane = t & 63;
  bool packed[kPlaceSlots];
  int c[kPlaceSlots];
  float v[kPlaceSlots];
#pragma unroll
  for (int k = 0; k < kPlaceSlots; ++k) {
    packed[k] = false;
    c[k] = J.f16 ? slot_column(slot0 + k, J.nrhs, packed[k]) : slot0 + k;
    v[k] = j < J.b.ldh ? gather_rhs(J, j, c[k]) : 0.f;
  }
  if (J.f16) {
    bool pk;
    const int w = t >> 6, cw = slot_column(slot0 + w, J.nrhs, pk);
    unsigned mb = cw < J.nrhs && lane < kColmaxBlocks ? J.b.colmax[cw * kColmaxBlocks + lane] : 0u;
    for (int off = 32; off > 0; off >>= 1) mb = max(mb, (unsigned)__shfl_xor((int)mb, off, 64));
    if (lane == 0) se[w] = cw < J.nrhs ? column_exponent(__uint_as_float(mb)) : 0;
  }
  __syncthreads();
  if (j >= J.b.ldh) return;
#pragma unroll
  for (int k = 0; k < kPlaceSlots; ++k) {
    if (J.f16) split_rhs_at(J, j, slot0 + k, c[k], packed[k], se[k], v[k]);
    else J.b.Vp[rhs_at(c[k], j, J.b.ncp)] = v[k];
  }
}

}  // namespace gpl
