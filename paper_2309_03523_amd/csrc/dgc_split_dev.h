// Device helpers of the kernels that take fp32 products as sums of bf16 products on
// v_mfma_f32_32x32x16_bf16 (why that is exact enough, and the operand layouts: dgc_dense_split.hip).
#pragma once

#include "dgc_internal.h"

namespace dgc {
namespace split {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
typedef int intx4 __attribute__((ext_vector_type(4)));

constexpr int kFrag = 64;   // uint4 of one fragment part (32 rows x 16 k, one bf16 part)

__device__ __forceinline__ bf16x8 as_frag(uint4 u) { return __builtin_bit_cast(bf16x8, u); }
__device__ __forceinline__ float cut(float x) { return __uint_as_float(__float_as_uint(x) & 0xffff0000u); }
__device__ __forceinline__ uint32_t tops(float lo, float hi) {   // the upper halves of two words
  return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}
__device__ __forceinline__ uint32_t nearest(float lo, float hi) {   // two floats, each rounded to the nearest bf16 number
  const bf16x2 v = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ float bf_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

// x = p[0] + p[1] + p[2], exactly, for finite x: p[0] the bf16 number nearest to x, p[1] the one nearest to what is left,
// p[2] the rest (at most seven bits).  To the nearest, not cut off: the rests then have either sign and half the size, and
// what a product of parts leaves out has either sign, too.
// An infinity goes into the low part: that meets only the other operand's high part, which has the sign of the whole
// number and is zero where that is.  Its other parts are the smallest normal number of its sign, so that two infinities
// make one, too.
template <int N>    // N numbers, two a word of h, m and l
__device__ __forceinline__ void split_parts(const float (&x)[N], uint32_t (&h)[N / 2], uint32_t (&m)[N / 2], uint32_t (&l)[N / 2]) {
  float top = 0.f;
#pragma unroll
  for (int i = 0; i < N / 2; ++i) {
    const float x0 = x[2 * i], x1 = x[2 * i + 1];
    h[i] = nearest(x0, x1);
    const float m0 = x0 - bf_lo(h[i]), m1 = x1 - bf_hi(h[i]);
    m[i] = nearest(m0, m1);
    l[i] = tops(m0 - bf_lo(m[i]), m1 - bf_hi(m[i]));
    top = fmaxf(top, fmaxf(fabsf(x0), fabsf(x1)));
  }
  if (__builtin_expect(__any(top > 3.3895313892515355e38f), 0)) {   // the largest bf16 number: beyond it, x may round to infinity
    float a[N], b[N], c[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      a[i] = cut(x[i]);
      b[i] = x[i] - a[i];
      c[i] = b[i] - cut(b[i]);
      if (fabsf(x[i]) == __builtin_inff()) {
        a[i] = b[i] = copysignf(1.1754943508222875e-38f, x[i]);
        c[i] = x[i];
      }
    }
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      h[i] = tops(a[2 * i], a[2 * i + 1]);
      m[i] = tops(b[2 * i], b[2 * i + 1]);
      l[i] = tops(c[2 * i], c[2 * i + 1]);
    }
  }
}
__device__ __forceinline__ void split8(const float (&x)[8], uint4 (&p)[3]) {
  uint32_t h[4], m[4], l[4];
  split_parts(x, h, m, l);
  p[0] = make_uint4(h[0], h[1], h[2], h[3]);
  p[1] = make_uint4(m[0], m[1], m[2], m[3]);
  p[2] = make_uint4(l[0], l[1], l[2], l[3]);
}
__device__ __forceinline__ void split4(const float (&x)[4], uint2 (&p)[3]) {
  uint32_t h[2], m[2], l[2];
  split_parts(x, h, m, l);
  p[0] = make_uint2(h[0], h[1]);
  p[1] = make_uint2(m[0], m[1]);
  p[2] = make_uint2(l[0], l[1]);
}

// The product of one fragment each, the smallest part products first: the five small ones to `small`, the large one to
// c, which may be the same.  (The instruction cuts its sums off rather than rounding them; small sums of their own lose less.)
__device__ __forceinline__ void five(floatx16& small, const uint4 (&w)[3], const uint4 (&x)[3]) {
  const bf16x8 w0 = as_frag(w[0]), w1 = as_frag(w[1]), w2 = as_frag(w[2]);
  const bf16x8 x0 = as_frag(x[0]), x1 = as_frag(x[1]), x2 = as_frag(x[2]);
  small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w0, x2, small, 0, 0, 0);
  small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w2, x0, small, 0, 0, 0);
  small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1, x1, small, 0, 0, 0);
  small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w0, x1, small, 0, 0, 0);
  small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1, x0, small, 0, 0, 0);
}
__device__ __forceinline__ void six(floatx16& c, floatx16& small, const uint4 (&w)[3], const uint4 (&x)[3]) {
  five(small, w, x);
  c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(w[0]), as_frag(x[0]), c, 0, 0, 0);
}

__device__ __forceinline__ void put(uint4* frag, const float (&x)[8]) {
  uint4 p[3];
  split8(x, p);
#pragma unroll
  for (int q = 0; q < 3; ++q) frag[q * kFrag] = p[q];
}

// x scale = h + l, two half-precision numbers, each the nearest to what is left: 22 to 24 bits of x, or what is above the
// smallest half-precision number.  Returns the largest magnitude: above kHalfMost / scale, h is infinite.
constexpr float kHalfMost = 65504.f;
template <int N>    // N numbers, two a word of h and l
__device__ __forceinline__ float halve(const float (&x)[N], float scale, uint32_t (&h)[N / 2], uint32_t (&l)[N / 2]) {
  float top = 0.f;
#pragma unroll
  for (int i = 0; i < N / 2; ++i) {
    const float x0 = x[2 * i], x1 = x[2 * i + 1];
    const halfx2 a = {(_Float16)(x0 * scale), (_Float16)(x1 * scale)};
    const halfx2 b = {(_Float16)fmaf(x0, scale, -(float)a.x), (_Float16)fmaf(x1, scale, -(float)a.y)};
    h[i] = __builtin_bit_cast(uint32_t, a);
    l[i] = __builtin_bit_cast(uint32_t, b);
    top = fmaxf(top, fmaxf(fabsf(x0), fabsf(x1)));
  }
  return top;
}
__device__ __forceinline__ float halve8(const float (&x)[8], float scale, uint4 (&p)[2]) {
  uint32_t h[4], l[4];
  const float top = halve(x, scale, h, l);
  p[0] = make_uint4(h[0], h[1], h[2], h[3]);
  p[1] = make_uint4(l[0], l[1], l[2], l[3]);
  return top;
}
__device__ __forceinline__ halfx8 as_halves(uint4 u) { return __builtin_bit_cast(halfx8, u); }
__device__ __forceinline__ void three(floatx16& c, floatx16& small, const uint4 (&w)[2], const uint4 (&x)[2]) {
  small = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_halves(w[0]), as_halves(x[1]), small, 0, 0, 0);
  small = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_halves(w[1]), as_halves(x[0]), small, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_halves(w[0]), as_halves(x[0]), c, 0, 0, 0);
}

// A table that no kernel writes while it is read: the address space lets wave-uniform entries come through the
// scalar cache, apart from the vector memory operations (which retire in order).
template <class T>
__device__ __forceinline__ T table_entry(const T* table, int64_t i) {
  union {
    T entry;
    uint32_t word[sizeof(T) / 4];
  } r;
  const auto* p = (const __attribute__((address_space(4))) uint32_t*)(table + i);
#pragma unroll
  for (size_t k = 0; k < sizeof(T) / 4; ++k) r.word[k] = p[k];
  return r.entry;
}

}  // namespace split
}  // namespace dgc
