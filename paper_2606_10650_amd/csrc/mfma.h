// MFMA fragments for gfx950 (CDNA4), 32x32 output tiles, K = 16 per step.
//
// A fragment (32 x 16): lane l holds row l % 32 and the 8 k-values of lane half
// l / 32 (element e <-> k index 8 * (l / 32) + e).  B fragment (16 x 32): lane l
// holds column l % 32 and the same 8 k-values.  The product pairs element e of
// a lane half of A with element e of the same lane half of B, so any fixed
// assignment of (lane half, element) to k that A and B share gives the same sum.
// Output (32 x 32, 16 floats per lane): lane l holds column l % 32 and rows
// 8 * (r / 4) + 4 * (l / 32) + r % 4 for r = 0..15.
#pragma once
#include "dla_common.h"

namespace dla {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

template <typename Tin>
struct Frag;

// bfloat16 inputs: one v_mfma_f32_32x32x16_bf16 per K = 16 step.
template <>
struct Frag<bf16_t> {
  using T = bf16x8;
  __device__ static __forceinline__ T load(const bf16_t* p) {  // 8 consecutive values
    return *reinterpret_cast<const T*>(p);
  }
  __device__ static __forceinline__ T from_floats(const float* x) {
    T r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = (__bf16)x[e];
    return r;
  }
  __device__ static __forceinline__ T zero() {
    T r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = (__bf16)0.f;
    return r;
  }
  __device__ static __forceinline__ void mma(f32x16& acc, const T& a, const T& b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
  }
};

// float32 inputs: eight v_mfma_f32_32x32x2_f32 per K = 16 step (element e of
// each lane half is one K = 2 product).
template <>
struct Frag<float> {
  using T = f32x8;
  __device__ static __forceinline__ T load(const float* p) {
    const float4 a = reinterpret_cast<const float4*>(p)[0];
    const float4 b = reinterpret_cast<const float4*>(p)[1];
    T r;
    r[0] = a.x; r[1] = a.y; r[2] = a.z; r[3] = a.w;
    r[4] = b.x; r[5] = b.y; r[6] = b.z; r[7] = b.w;
    return r;
  }
  __device__ static __forceinline__ T from_floats(const float* x) {
    T r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = x[e];
    return r;
  }
  __device__ static __forceinline__ T zero() {
    T r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = 0.f;
    return r;
  }
  __device__ static __forceinline__ void mma(f32x16& acc, const T& a, const T& b) {
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], acc, 0, 0, 0);
  }
};

// 16 x 16 output tiles, K = 32 per step: lane l holds row (A) or column (B)
// l % 16 and 8 k-values, the k set being the lane quarter's; as above, any
// assignment of (lane quarter, element) to k that A and B share gives the same
// sum.  Output: lane l holds column l % 16 and rows 4 (l / 16) + r, r = 0..3.
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void mma16(f32x4& acc, const bf16x8& a, const bf16x8& b) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ void mma16(f32x4& acc, const f32x8& a, const f32x8& b) {
#pragma unroll
  for (int e = 0; e < 8; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], acc, 0, 0, 0);
}
// float64 16 x 16 tiles, K = 16 per call: step r takes the k set 4 r + l / 16, and
// lane l holds row (A) or column (B) l % 16; output: column l % 16 and rows 4 r + l
// / 16, so that a result serves as the next product's B operand.
typedef double f64x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void mma16(f64x4& acc, const f64x4& a, const f64x4& b) {
#pragma unroll
  for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r], b[r], acc, 0, 0, 0);
}
// The tile's K = 32 product of the inputs, summed in float64: bfloat16 operands by
// bfloat16 MFMAs over 16 products each (exact products, one float32 sum), which
// takes half the time of float64 MFMAs; float32 operands by float64 MFMAs.
// gram_row: the output row of element r.
__device__ __forceinline__ void gram16(f64x4& acc, const bf16x8& a, const bf16x8& b) {
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  const s16x8 x = __builtin_bit_cast(s16x8, a), y = __builtin_bit_cast(s16x8, b);
  f32x4 z0 = {0.f, 0.f, 0.f, 0.f}, z1 = z0;
  z0 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_shufflevector(x, x, 0, 1, 2, 3),
                                                 __builtin_shufflevector(y, y, 0, 1, 2, 3), z0, 0, 0, 0);
  z1 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_shufflevector(x, x, 4, 5, 6, 7),
                                                 __builtin_shufflevector(y, y, 4, 5, 6, 7), z1, 0, 0, 0);
#pragma unroll
  for (int r = 0; r < 4; ++r) acc[r] += (double)z0[r] + (double)z1[r];
}
__device__ __forceinline__ void gram16(f64x4& acc, const f32x8& a, const f32x8& b) {
#pragma unroll
  for (int e = 0; e < 8; ++e)
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[e], (double)b[e], acc, 0, 0, 0);
}
template <typename Tin>
__device__ __forceinline__ int gram_row(int r, int q4) {
  return sizeof(Tin) == 2 ? 4 * q4 + r : 4 * r + q4;
}

// A float32 operand as three bfloat16 terms, largest first, whose sum is its
// value to float32 rounding.
struct Split3 {
  bf16x8 t[3];
  __device__ __forceinline__ explicit Split3(const f32x8& x) {
    f32x8 y = x;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        t[q][e] = (__bf16)y[e];
        y[e] -= (float)t[q][e];
      }
    }
  }
};
// acc += a b to float32 rounding: float32 operands by float32 MFMAs, or, with
// the bfloat16 rate, by the six products of their terms that matter (the
// smallest first); b exact in bfloat16 takes three.
__device__ __forceinline__ void mma16_split(f32x4& acc, const Split3& a, const Split3& b) {
  mma16(acc, a.t[2], b.t[0]);
  mma16(acc, a.t[0], b.t[2]);
  mma16(acc, a.t[1], b.t[1]);
  mma16(acc, a.t[1], b.t[0]);
  mma16(acc, a.t[0], b.t[1]);
  mma16(acc, a.t[0], b.t[0]);
}
__device__ __forceinline__ void mma16_split(f32x4& acc, const Split3& a, const bf16x8& b) {
#pragma unroll
  for (int q = 2; q >= 0; --q) mma16(acc, a.t[q], b);
}
__device__ __forceinline__ void mma16_split(f32x4& acc, const bf16x8& a, const Split3& b) {
#pragma unroll
  for (int q = 2; q >= 0; --q) mma16(acc, a, b.t[q]);
}

__device__ __forceinline__ f32x16 zero16() {
  f32x16 r;
#pragma unroll
  for (int i = 0; i < 16; ++i) r[i] = 0.f;
  return r;
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));  // 16 bytes, first-class
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// element e of a 16-byte piece of elements of type Tin
template <typename Tin>
__device__ __forceinline__ Tin piece_elem(const u32x4& v, int e);
template <>
__device__ __forceinline__ bf16_t piece_elem<bf16_t>(const u32x4& v, int e) {
  bf16_t r;
  r.x = static_cast<uint16_t>(v[e >> 1] >> (16 * (e & 1)));
  return r;
}
template <>
__device__ __forceinline__ float piece_elem<float>(const u32x4& v, int e) {
  return __uint_as_float(v[e]);
}

// 8 operand values from two runs of 4 consecutive elements (each run aligned
// to 4 elements)
template <typename Tin>
__device__ __forceinline__ typename Frag<Tin>::T load_4x2(const Tin* p0, const Tin* p1);
template <>
__device__ __forceinline__ bf16x8 load_4x2<bf16_t>(const bf16_t* p0, const bf16_t* p1) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  const bf16x4 lo = *reinterpret_cast<const bf16x4*>(p0);
  const bf16x4 hi = *reinterpret_cast<const bf16x4*>(p1);
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
template <>
__device__ __forceinline__ f32x8 load_4x2<float>(const float* p0, const float* p1) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const f32x4 lo = *reinterpret_cast<const f32x4*>(p0);
  const f32x4 hi = *reinterpret_cast<const f32x4*>(p1);
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// 4 consecutive elements as floats (8-byte aligned for bfloat16, 16 for float32)
__device__ __forceinline__ void load4f(const bf16_t* p, float (&x)[4]) {
  const uint2 u = *reinterpret_cast<const uint2*>(p);
  x[0] = __uint_as_float(u.x << 16);
  x[1] = __uint_as_float(u.x & 0xFFFF0000u);
  x[2] = __uint_as_float(u.y << 16);
  x[3] = __uint_as_float(u.y & 0xFFFF0000u);
}
__device__ __forceinline__ void load4f(const float* p, float (&x)[4]) {
  const float4 v = *reinterpret_cast<const float4*>(p);
  x[0] = v.x;
  x[1] = v.y;
  x[2] = v.z;
  x[3] = v.w;
}

// row (within the 32-row tile) of output element r held by lane l
__device__ __forceinline__ int out_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

}  // namespace dla
