// Device-side helpers shared by the kernels: storage types, conversions, wave reductions.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"

namespace mk {

typedef uint16_t bf16_t;   // raw bfloat16 bits

__device__ __forceinline__ float bf16_to_f32(bf16_t v) {
  return __uint_as_float(((uint32_t)v) << 16);
}
// round to nearest, ties to even: the hardware conversion of gfx950 (v_cvt_pk_bf16_f32)
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  return __builtin_bit_cast(bf16_t, (__bf16)f);
}
// two values in one conversion: a in the low half, b in the high half
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const f32x2_t v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// rows of sample b: the first, how many there are, how many of them may be attended to
struct Sample { int64_t first; int n, keys; };
__device__ __forceinline__ Sample sample_rows(const Rows& r, int b, int L) {
  const int keys = r.lens ? r.lens[b] : L;
  if (!r.ends) return {(int64_t)b * L, L, keys};
  const int first = b ? r.ends[b - 1] : r.first;
  return {first - r.first, r.ends[b] - first, keys};
}

// row of the padded batch that row `row` stands for
__device__ __forceinline__ int padded_row(const Rows& r, int row, int B, int L) {
  if (!r.ends) return row;
  int lo = 0, hi = B - 1;                             // the first sample that ends behind the row
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (r.ends[mid] > row) hi = mid; else lo = mid + 1;
  }
  return lo * L + row - (lo ? r.ends[lo - 1] : 0);
}

template <typename T> __device__ __forceinline__ float ld(const T* p);
template <> __device__ __forceinline__ float ld<float>(const float* p) { return *p; }
template <> __device__ __forceinline__ float ld<bf16_t>(const bf16_t* p) { return bf16_to_f32(*p); }

template <typename T> __device__ __forceinline__ void st(T* p, float v);
template <> __device__ __forceinline__ void st<float>(float* p, float v) { *p = v; }
template <> __device__ __forceinline__ void st<bf16_t>(bf16_t* p, float v) { *p = f32_to_bf16(v); }

// value a T would hold after a store (used where a kernel must behave as if it re-read its output)
template <typename T> __device__ __forceinline__ float rnd(float v);
template <> __device__ __forceinline__ float rnd<float>(float v) { return v; }
template <> __device__ __forceinline__ float rnd<bf16_t>(float v) { return bf16_to_f32(f32_to_bf16(v)); }

// Sums (maxima) over the 64 lanes of a wave, the result in every lane.  Inside a row of 16 lanes
// four rotating DPP adds (by 8, 4, 2, 1) leave the row's total in each of its lanes; the four
// rows are then read through scalar registers and combined in row order.  A butterfly of
// cross-lane shuffles costs six dependent trips through the LDS crossbar instead, which is what
// the row-wise kernels spent most of their time on.  The order of the additions is fixed.
template <int CTRL>
__device__ __forceinline__ float dpp_rotate(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float lane_value(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_rotate<0x128>(v);   // row_ror:8
  v += dpp_rotate<0x124>(v);   // row_ror:4
  v += dpp_rotate<0x122>(v);   // row_ror:2
  v += dpp_rotate<0x121>(v);   // row_ror:1
  return ((lane_value(v, 0) + lane_value(v, 16)) + lane_value(v, 32)) + lane_value(v, 48);
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_rotate<0x128>(v));
  v = fmaxf(v, dpp_rotate<0x124>(v));
  v = fmaxf(v, dpp_rotate<0x122>(v));
  v = fmaxf(v, dpp_rotate<0x121>(v));
  return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)), fmaxf(lane_value(v, 32), lane_value(v, 48)));
}

__device__ __forceinline__ float gelu_erf(float x) {
  return 0.5f * x * (1.0f + erff(x * 0.70710678118654752440f));
}
// GELU where the result is rounded to bf16.  The tile store of a feed-forward product evaluates it
// once per output on a unit that does nothing else meanwhile, so its instructions are the product's
// time: no divisions, constants folded, and the half of each function that tends to zero is the one
// computed, so that nothing cancels (largest error against 64 bits over |x| < 9 before the rounding:
// 3.3e-7 for the erf form, 4.7e-7 with a division and 1 + erf).
// 16384 x 4096 outputs of K = 1024, erf form: 187 -> 176 us; 6352 x 4096 85 -> 80; 6400 x 3072 60 -> 58.
//
// half_erfc = erfc(|x| / sqrt 2) / 2 by the rational approximation of Abramowitz & Stegun 7.1.26
// (absolute error < 0.75e-7); density = exp(-x^2 / 2), the approximation's own exponential
__device__ __forceinline__ float half_erfc(float x, float& density) {
  const float d = fmaf(0.3275911f * 0.70710678118654752440f, fabsf(x), 1.0f), r = __builtin_amdgcn_rcpf(d);
  const float t = fmaf(fmaf(-d, r, 1.0f), r, r);      // one Newton step: as good as a division
  density = __builtin_amdgcn_exp2f(x * x * (-0.5f * 1.44269504088896340736f));
  float p = fmaf(t, 0.5f * 1.061405429f, 0.5f * -1.453152027f);
  p = fmaf(t, p, 0.5f * 1.421413741f);
  p = fmaf(t, p, 0.5f * -0.284496736f);
  p = fmaf(t, p, 0.5f * 0.254829592f);
  return p * t * density;
}
__device__ __forceinline__ float gelu_erf_bf16(float x) {
  float density;
  const float ax = fminf(fabsf(x), 64.0f);            // keeps infinities out of the product; both terms see NaN
  return fmaf(-ax, half_erfc(ax, density), 0.5f * (x + fabsf(x)));
}
// tanh form: 0.5 (1 - tanh |u|) = 1 / (1 + exp(2|u|)), exact limits at both ends
__device__ __forceinline__ float half_tanhc(float x) {
  const float c = 2.0f * 0.79788456080286535588f * 1.44269504088896340736f;
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(fabsf(x) * fmaf(c * 0.044715f, x * x, c)));
}
__device__ __forceinline__ float gelu_tanh_bf16(float x) {
  const float ax = fminf(fabsf(x), 64.0f);
  return fmaf(-ax, half_tanhc(ax), 0.5f * (x + fabsf(x)));
}
__device__ __forceinline__ float gelu_tanh(float x) {
  const float c = 0.79788456080286535588f;
  return 0.5f * x * (1.0f + tanhf(c * (x + 0.044715f * x * x * x)));
}
__device__ __forceinline__ float gelu_erf_grad(float x) {
  float cdf = 0.5f * (1.0f + erff(x * 0.70710678118654752440f));
  float pdf = 0.39894228040143267794f * __expf(-0.5f * x * x);
  return cdf + x * pdf;
}
// the derivatives where the result is rounded to bf16
__device__ __forceinline__ float gelu_erf_grad_bf16(float x) {
  float density;
  const float q = half_erfc(x, density);
  return fmaf(x * 0.39894228040143267794f, density, 0.5f + copysignf(0.5f - q, x));
}
__device__ __forceinline__ float gelu_tanh_grad_bf16(float x) {
  const float c = 2.0f * 0.79788456080286535588f, h = half_tanhc(x);
  return fmaf(fmaf(-h, h, h) * x, fmaf(3.0f * 0.044715f * c, x * x, c), 0.5f + copysignf(0.5f - h, x));
}
__device__ __forceinline__ float gelu_tanh_grad(float x) {
  const float c = 0.79788456080286535588f;
  float t = tanhf(c * (x + 0.044715f * x * x * x));
  return 0.5f * (1.0f + t) + 0.5f * x * (1.0f - t * t) * c * (1.0f + 0.134145f * x * x);
}

}  // namespace mk
