// Internal helpers shared by the gplens translation units: error reporting,
// workspace carving, launch checks and small device utilities.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstddef>
#include <cstdint>
#include <cstdio>

#include "../../include/gplens.h"

namespace gpl {

// Last error text, per host thread.
void set_error(const char* fmt, ...);
const char* last_error();

#define GPL_REQUIRE(cond, ...)              \
  do {                                      \
    if (!(cond)) {                          \
      ::gpl::set_error(__VA_ARGS__);        \
      return GPL_EINVAL;                    \
    }                                       \
  } while (0)

#define GPL_HIP(call)                                                                        \
  do {                                                                                       \
    hipError_t e_ = (call);                                                                  \
    if (e_ != hipSuccess) {                                                                  \
      ::gpl::set_error("%s:%d %s: %s", __FILE__, __LINE__, #call, hipGetErrorString(e_));    \
      return GPL_EHIP;                                                                       \
    }                                                                                        \
  } while (0)

#define GPL_LAUNCH_CHECK() GPL_HIP(hipGetLastError())

#define GPL_TRY(expr)     \
  do {                    \
    int rc_ = (expr);     \
    if (rc_ != GPL_OK) return rc_; \
  } while (0)

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x, size_t a = kAlign) { return (x + a - 1) / a * a; }
__host__ __device__ inline int round_up(int x, int m) { return (x + m - 1) / m * m; }
__host__ __device__ inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// Bump allocator over a caller-provided workspace. `take` returns nullptr when
// the workspace is exhausted (callers check `ok()` once after carving).
struct Carver {
  char* base;
  size_t cap;
  size_t used = 0;
  bool overflow = false;
  Carver(void* ws, size_t bytes) : base(static_cast<char*>(ws)), cap(bytes) {}
  template <class T>
  T* take(size_t count) {
    size_t off = align_up(used);
    size_t need = off + align_up(count * sizeof(T));
    if (base == nullptr || need > cap) {
      overflow = true;
      used = need;
      return nullptr;
    }
    used = need;
    return reinterpret_cast<T*>(base + off);
  }
  bool ok() const { return !overflow; }
};

// Size-only pass of the same carving sequence.
struct Sizer {
  size_t used = 0;
  template <class T>
  T* take(size_t count) {
    used = align_up(used) + align_up(count * sizeof(T));
    return nullptr;
  }
};

inline int check_ws(void* ws, size_t have, size_t need) {
  if (need == 0) return GPL_OK;
  if (ws == nullptr || (reinterpret_cast<uintptr_t>(ws) % kAlign) != 0) {
    set_error("workspace must be non-NULL and %zu-byte aligned", kAlign);
    return GPL_EWORKSPACE;
  }
  if (have < need) {
    set_error("workspace too small: %zu bytes given, %zu needed", have, need);
    return GPL_EWORKSPACE;
  }
  return GPL_OK;
}

// ---- device helpers

__device__ inline float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// v of the lane whose index differs in bit OFF (32 ... 1), where OFF = 4 asks that lanes
// differing in bit 3 hold the same value: DPP moves within rows of 16 lanes, permlane
// swaps across them, no trip through LDS.
template <int OFF>
__device__ __forceinline__ unsigned lane_xor(unsigned v) {
  if constexpr (OFF == 32) {
    const auto s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (threadIdx.x & 32) ? s[0] : s[1];
  } else if constexpr (OFF == 16) {
    const auto s = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return (threadIdx.x & 16) ? s[0] : s[1];
  } else {
    constexpr int ctrl = OFF == 8 ? 0x128 : OFF == 4 ? 0x124 : OFF == 2 ? 0x4e : 0xb1;  // row_ror:8, :4, quad_perm
    return (unsigned)__builtin_amdgcn_mov_dpp((int)v, ctrl, 0xf, 0xf, true);
  }
}
template <int OFF, class T>
__device__ __forceinline__ T add_lane_xor(T v) {
  static_assert(sizeof(T) == 4 || sizeof(T) == 8, "a register or two");
  if constexpr (sizeof(T) == 4) {
    return v + __builtin_bit_cast(T, lane_xor<OFF>(__builtin_bit_cast(unsigned, v)));
  } else {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned long long o =
        ((unsigned long long)lane_xor<OFF>((unsigned)(b >> 32)) << 32) | lane_xor<OFF>((unsigned)b);
    return v + __builtin_bit_cast(T, o);
  }
}

// Sum over the wave, the same in every lane (a butterfly from the widest step down).
template <class T>
__device__ __forceinline__ T warp_sum(T v) {
  v = add_lane_xor<32>(v);
  v = add_lane_xor<16>(v);
  v = add_lane_xor<8>(v);
  v = add_lane_xor<4>(v);
  v = add_lane_xor<2>(v);
  return add_lane_xor<1>(v);
}

// Inclusive prefix sum over the wave in lane order, every lane active: shifts within rows
// of 16 lanes, then the rows' last lanes broadcast onwards.
__device__ __forceinline__ int warp_prefix(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2, 3
  return v;
}

// Largest of the wave's values, the same in every lane.
__device__ __forceinline__ float warp_max(float v) {
  auto step = [](float a, unsigned b) { return fmaxf(a, __builtin_bit_cast(float, b)); };
  v = step(v, lane_xor<32>(__builtin_bit_cast(unsigned, v)));
  v = step(v, lane_xor<16>(__builtin_bit_cast(unsigned, v)));
  v = step(v, lane_xor<8>(__builtin_bit_cast(unsigned, v)));
  v = step(v, lane_xor<4>(__builtin_bit_cast(unsigned, v)));
  v = step(v, lane_xor<2>(__builtin_bit_cast(unsigned, v)));
  return step(v, lane_xor<1>(__builtin_bit_cast(unsigned, v)));
}

// Sum of p[0, cnt) over the 64 lanes of one wave in a fixed order (lane-strided
// partial sums, then a butterfly); the result is the same in every lane.
__device__ inline double wave_fold_sum(const double* __restrict__ p, int cnt) {
  double s = 0.0;
  for (int k = (int)(threadIdx.x & 63); k < cnt; k += 64) s += p[k];
  return warp_sum(s);
}

// Deterministic block reduction of one double per thread (blockDim.x <= 1024,
// multiple of 64). Result valid in thread 0.
__device__ inline double block_sum_double(double v, double* smem) {
  v = warp_sum(v);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if (lane == 0) smem[wid] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < nw; ++w) s += smem[w];
  return s;
}

// Kernel scaling: exp(-d^2 / (2 l^2)) = exp2(-d^2 * kscale2), kscale2 = log2(e)/(2 l^2).
inline double kernel_scale2(double lengthscale) { return 1.4426950408889634 / (2.0 * lengthscale * lengthscale); }

}  // namespace gpl
