// Matrix-core operands of the scoring kernels: the 32x32 MFMA of each query
// dtype, its fragments, and the element operations on them (gfx950).
#pragma once

#include "pk_device.h"

namespace pk {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

// Lambdas of the scoring kernels are always inlined: register arrays indexed
// by their arguments must see those arguments as constants.
#define PK_INLINE __attribute__((always_inline))

template <typename T>
struct MfmaOp;

template <>
struct MfmaOp<uint16_t> {  // bf16 storage
  static constexpr int KSTEP = 16;  // reduction elements per instruction
  static constexpr int LANE_K = 8;  // reduction elements supplied per lane
  static constexpr int ESIZE = 2;
  using frag = bf16x8_t;
  __device__ static __forceinline__ f32x16_t mma(frag a, frag b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
  __device__ static __forceinline__ frag load(const void* p) {
    return __builtin_bit_cast(frag, *reinterpret_cast<const uint4*>(p));
  }
  __device__ static __forceinline__ frag zero() { return __builtin_bit_cast(frag, uint4{0, 0, 0, 0}); }
  __device__ static __forceinline__ float to_f32(uint16_t v) { return bf16_to_f32(v); }
  __device__ static __forceinline__ float stored(float v) { return round_bf16_f32(v); }
  // sum over the fragment's 8 elements of f[i] * s[i] (s: 8 bf16, 16-byte aligned)
  __device__ static __forceinline__ float dot(frag f, const uint16_t* s) {
    const uint4 u = __builtin_bit_cast(uint4, f);
    const uint4 v = *reinterpret_cast<const uint4*>(s);
    float a = bf16_lo(u.x) * bf16_lo(v.x);
    a = fmaf(bf16_hi(u.x), bf16_hi(v.x), a);
    a = fmaf(bf16_lo(u.y), bf16_lo(v.y), a);
    a = fmaf(bf16_hi(u.y), bf16_hi(v.y), a);
    a = fmaf(bf16_lo(u.z), bf16_lo(v.z), a);
    a = fmaf(bf16_hi(u.z), bf16_hi(v.z), a);
    a = fmaf(bf16_lo(u.w), bf16_lo(v.w), a);
    return fmaf(bf16_hi(u.w), bf16_hi(v.w), a);
  }
  // Normalised fragment, rounded to bf16 (nearest, ties to even).
  __device__ static __forceinline__ frag normalize(frag f, float mean, float rstd) {
    uint4 u = __builtin_bit_cast(uint4, f);
    u.x = pack_bf16x2(qn_apply(bf16_lo(u.x), mean, rstd), qn_apply(bf16_hi(u.x), mean, rstd));
    u.y = pack_bf16x2(qn_apply(bf16_lo(u.y), mean, rstd), qn_apply(bf16_hi(u.y), mean, rstd));
    u.z = pack_bf16x2(qn_apply(bf16_lo(u.z), mean, rstd), qn_apply(bf16_hi(u.z), mean, rstd));
    u.w = pack_bf16x2(qn_apply(bf16_lo(u.w), mean, rstd), qn_apply(bf16_hi(u.w), mean, rstd));
    return __builtin_bit_cast(frag, u);
  }
};

template <>
struct MfmaOp<float> {
  static constexpr int KSTEP = 2;
  static constexpr int LANE_K = 1;
  static constexpr int ESIZE = 4;
  using frag = float;
  __device__ static __forceinline__ f32x16_t mma(frag a, frag b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
  __device__ static __forceinline__ frag load(const void* p) { return *reinterpret_cast<const float*>(p); }
  __device__ static __forceinline__ frag zero() { return 0.f; }
  __device__ static __forceinline__ float to_f32(float v) { return v; }
  __device__ static __forceinline__ float stored(float v) { return v; }
  __device__ static __forceinline__ frag normalize(frag f, float mean, float rstd) {
    return qn_apply(f, mean, rstd);
  }
};

// Row of the 32x32 MFMA result held in accumulator slot j of a lane whose
// upper-half bit is kh (columns are lane & 31).
__device__ __forceinline__ int acc_row(int j, int kh) { return 8 * (j >> 2) + 4 * kh + (j & 3); }

}  // namespace pk
