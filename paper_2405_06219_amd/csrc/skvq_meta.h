// Storage formats of (scale, zero) (Section 4.1: FP8 E4M3; Section 4.3 also counts fp16), device
// side.  A pair is stored scale first; element size 4, 2 or 1 byte.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "skvq.h"

namespace skvq {

// Two floats -> FP8 E4M3 (bias 7, largest finite value 448): nearest, ties to even, saturating (a NaN
// of either sign, which finite inputs do not lead to, is 448); the first in the low byte.  One conversion
// instruction on values that its saturation mode does not concern; for every float that is no NaN it gives
// the number that rounding with integer arithmetic does, which takes forty instructions per pair.
__device__ __forceinline__ unsigned e4m3_pair(float a, float b) {
  return (unsigned)__builtin_amdgcn_cvt_pk_fp8_f32(fmaxf(fminf(a, 448.0f), -448.0f), fmaxf(fminf(b, 448.0f), -448.0f),
                                                   0, false) & 0xffffu;
}

// FP8 E4M3 -> float, exact (NaN encodings are never stored).
__device__ __forceinline__ float e4m3_to_float(unsigned b) {
  const unsigned e = (b >> 3) & 15u, m = b & 7u;
  const float v = e ? __uint_as_float(((e + 120u) << 23) | (m << 20)) : (float)m * 0.001953125f;
  return (b & 0x80u) ? -v : v;
}

// A (scale, zero) pair as it reads back from storage, and its storage word (fp16: scale in the
// low half; FP8: scale in the low byte; unused for fp32).
struct MetaPair {
  float scale, zero;
  unsigned stored;
};

__device__ __forceinline__ MetaPair meta_make(float scale, float zero, int fmt) {
  MetaPair m;
  if (fmt == SKVQ_META_F16) {
    const __half2 h = __halves2half2(__float2half_rn(scale), __float2half_rn(zero));
    m.scale = __low2float(h);
    m.zero = __high2float(h);
    m.stored = __builtin_bit_cast(unsigned, h);
  } else if (fmt == SKVQ_META_FP8_E4M3) {
    m.stored = e4m3_pair(scale, zero);
    m.scale = __builtin_amdgcn_cvt_f32_fp8((int)m.stored, 0);  // decoding is exact
    m.zero = __builtin_amdgcn_cvt_f32_fp8((int)m.stored, 1);
  } else {
    m.scale = scale;
    m.zero = zero;
    m.stored = 0;
  }
  return m;
}

__device__ __forceinline__ void meta_store_pair(void *base, long long pair, const MetaPair &m, int fmt) {
  if (fmt == SKVQ_META_F16)
    reinterpret_cast<unsigned *>(base)[pair] = m.stored;
  else if (fmt == SKVQ_META_FP8_E4M3)
    reinterpret_cast<unsigned short *>(base)[pair] = (unsigned short)m.stored;
  else
    reinterpret_cast<float2 *>(base)[pair] = make_float2(m.scale, m.zero);
}

__device__ __forceinline__ float2 meta_load_pair(const void *base, long long pair, int fmt) {
  if (fmt == SKVQ_META_F16) {
    const __half2 h = reinterpret_cast<const __half2 *>(base)[pair];
    return make_float2(__low2float(h), __high2float(h));
  }
  if (fmt == SKVQ_META_FP8_E4M3) {
    const unsigned w = reinterpret_cast<const unsigned short *>(base)[pair];
    return make_float2(e4m3_to_float(w & 0xffu), e4m3_to_float(w >> 8));
  }
  return reinterpret_cast<const float2 *>(base)[pair];
}

}  // namespace skvq
