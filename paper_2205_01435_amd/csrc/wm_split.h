// fp32 products on the bf16 matrix unit from exact three-term splits.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wm_device.h"

namespace wm {

// ---------------------------------------------------------------------------
// fp32 products on the bf16 matrix unit.  A float is the exact sum of three
// bf16 values, x = h + m + l (8 significant bits each, rounded to nearest, so
// that the signs carry the rest: |m| <= 2^-8 |x|, |l| <= 2^-17 |x|), and six
// of the nine products of two such sums, accumulated in fp32, leave out only
// m l + l m + l l, at most about 2^-24 of the product: as much as the rounding
// of one fp32 product.  At 16 times the fp32 MFMA rate the six cost 3/8
// of the fp32 instruction's time.  Error against 64 bits of a K 512 dot
// product (uniform operands, fp32 accumulation either way): 3.3e-7 of the
// result's norm, 4.1e-7 with the fp32 MFMA; K 1056 4.9e-7 and 5.8e-7.
// An infinity, or a finite value above the largest bf16, becomes NaN (inf - inf
// in the remainder), in every sum that it enters; NaN stays NaN.  The kernels
// take the sums that came out as NaN again on the fp32 unit (nan_to).
// ---------------------------------------------------------------------------
struct Split3 {
  bf16x8 h, m, l;
};

// the eight floats of two 16-byte pieces
__device__ __forceinline__ Split3 split3(const float (&x)[8]) {
  uint32_t h[4], m[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h[i] = pack2_bf16(x[2 * i], x[2 * i + 1]);
    const float r0 = x[2 * i] - __uint_as_float(h[i] << 16);
    const float r1 = x[2 * i + 1] - __uint_as_float(h[i] & 0xffff0000u);
    m[i] = pack2_bf16(r0, r1);
    l[i] = pack2_bf16(r0 - __uint_as_float(m[i] << 16), r1 - __uint_as_float(m[i] & 0xffff0000u));
  }
  return Split3{__builtin_bit_cast(bf16x8, make_uint4(h[0], h[1], h[2], h[3])),
                __builtin_bit_cast(bf16x8, make_uint4(m[0], m[1], m[2], m[3])),
                __builtin_bit_cast(bf16x8, make_uint4(l[0], l[1], l[2], l[3]))};
}
__device__ __forceinline__ Split3 split3(uint4 u, uint4 v) {
  const float x[8] = {__uint_as_float(u.x), __uint_as_float(u.y), __uint_as_float(u.z), __uint_as_float(u.w),
                      __uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w)};
  return split3(x);
}

__device__ __forceinline__ bool any_nan(f32x4 v) {
  return v[0] != v[0] || v[1] != v[1] || v[2] != v[2] || v[3] != v[3];
}
// v with the elements that are NaN from w
__device__ __forceinline__ f32x4 nan_to(f32x4 v, f32x4 w) {
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = v[i] != v[i] ? w[i] : v[i];
  return v;
}

__device__ __forceinline__ f32x4 mfma_bf16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// acc[i] += a[i] . b over one 32-wide K slice for N fragments a against one b:
// the small products first, the N independent accumulators interleaved
template <int N>
__device__ __forceinline__ void mfma_split(f32x4 (&acc)[N], const Split3 (&a)[N], const Split3& b) {
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf16(a[i].m, b.m, acc[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf16(a[i].l, b.h, acc[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf16(a[i].h, b.l, acc[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf16(a[i].m, b.h, acc[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf16(a[i].h, b.m, acc[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf16(a[i].h, b.h, acc[i]);
}

}  // namespace wm
