// Shared device helpers for librattn (gfx950 only: 64-wide wavefronts).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "kernels.hpp"

namespace rattn {

typedef uint16_t bf16_t;  // raw bfloat16 bits

__device__ __forceinline__ float bf16_to_f32(bf16_t x) { return __uint_as_float(((uint32_t)x) << 16); }

// round-to-nearest-even; NaN stays NaN
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

template <typename IO> struct io_traits;

template <> struct io_traits<float> {
  static __device__ __forceinline__ float ld(const float* p) { return *p; }
  static __device__ __forceinline__ void st(float* p, float v) { *p = v; }
};

template <> struct io_traits<bf16_t> {
  static __device__ __forceinline__ float ld(const bf16_t* p) { return bf16_to_f32(*p); }
  static __device__ __forceinline__ void st(bf16_t* p, float v) { *p = f32_to_bf16(v); }
};

// Reductions over lanes that stay in registers (DPP within 16 lanes, permlane swaps across): every lane gets the result.
template <int CTRL>
__device__ __forceinline__ float dpp_get(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), CTRL, 0xf, 0xf, false));
}
template <typename F> __device__ __forceinline__ float row16_reduce(float x, F f) {
  x = f(x, dpp_get<0xB1>(x));     // quad_perm [1,0,3,2]
  x = f(x, dpp_get<0x4E>(x));     // quad_perm [2,3,0,1]
  x = f(x, dpp_get<0x141>(x));    // row_half_mirror
  return f(x, dpp_get<0x140>(x)); // row_mirror
}
// across the four 16-lane rows of a wave (lanes l, l^16, l^32, l^48)
template <typename F> __device__ __forceinline__ float rows_reduce(float x, F f) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = f(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return f(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float rows_sum(float x) { return rows_reduce(x, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float rows_max(float x) { return rows_reduce(x, [](float a, float b) { return fmaxf(a, b); }); }
__device__ __forceinline__ float sum16(float x) { return row16_reduce(x, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float sum8(float x) {  // over 8 consecutive lanes
  x += dpp_get<0xB1>(x);
  x += dpp_get<0x4E>(x);
  return x + dpp_get<0x141>(x);
}
__device__ __forceinline__ float wave_sum(float x) { return rows_sum(sum16(x)); }
__device__ __forceinline__ float wave_max(float x) { return rows_max(row16_reduce(x, [](float a, float b) { return fmaxf(a, b); })); }
// Feature map of the linear branch: softmax over the features (Sec. 3.1), or the ablation's ReLU / identity
// (Sec. 4.5).  Every map is written phi(x)[f] = feat(x[f], m) / z with row statistics (m, z): the row maximum and
// the sum of exponentials for softmax, (0, 1) for the other two.  `phi` is uniform over a launch.
__device__ __forceinline__ float feat(float x, float m, int phi) {
  if (phi == PHI_SOFTMAX) return expf(x - m);
  return phi == PHI_RELU ? fmaxf(x, 0.f) : x;
}
// phi of a row of 64*EPL features spread over the wave (element d in lane d % 64, register d / 64)
template <int EPL>
__device__ __forceinline__ void feature_row(const float (&x)[EPL], float (&f)[EPL], int phi) {
  if (phi == PHI_SOFTMAX) {
    float m = x[0];
#pragma unroll
    for (int e = 1; e < EPL; ++e) m = fmaxf(m, x[e]);
    m = wave_max(m);
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) { f[e] = expf(x[e] - m); s += f[e]; }
    s = 1.f / wave_sum(s);
#pragma unroll
    for (int e = 0; e < EPL; ++e) f[e] *= s;
  } else {
#pragma unroll
    for (int e = 0; e < EPL; ++e) f[e] = phi == PHI_RELU ? fmaxf(x[e], 0.f) : x[e];
  }
}
// Tile `i` of a DgammaSum, by 256 threads: 32 consecutive (head, feature) entries of one of the two gains.  Thread
// (rg = tid / 8, c = tid % 8) adds every 32nd partial starting at rg for entries 4c .. 4c+3 (independent 16-byte loads),
// then the 32 sums are added in order.
__device__ __forceinline__ void dgamma_reduce_tile(const DgammaSum& dg, int i) {
  __shared__ float4 part[32][8];
  const int half = dg.HD / 32, which = i / half, rg = threadIdx.x >> 3, c = threadIdx.x & 7;
  float* out = which == 0 ? dg.dgs : which == 1 ? dg.dgr : nullptr;
  if (!out) return;   // (block-uniform)
  const int e = (i % half) * 32 + 4 * c;
  const float* src = dg.part + (size_t)which * dg.RB * dg.HD + e;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
  for (int r = rg; r < dg.RB; r += 32) {
    const float4 x = *reinterpret_cast<const float4*>(src + (size_t)r * dg.HD);
    s.x += x.x; s.y += x.y; s.z += x.z; s.w += x.w;
  }
  part[rg][c] = s;
  __syncthreads();
  if (rg == 0) {
    float4 t = part[0][c];
#pragma unroll
    for (int j = 1; j < 32; ++j) { const float4 x = part[j][c]; t.x += x.x; t.y += x.y; t.z += x.z; t.w += x.w; }
    *reinterpret_cast<float4*>(out + e) = t;
  }
}
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }
__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63); }

}  // namespace rattn
