// fp32 products on the bf16 matrix cores: exact splitting of floats into three
// bfloat16 parts, shared by the channel contraction and the matrix transforms
// (after Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations", ARITH 2019).
#pragma once

#include <hip/hip_runtime.h>

namespace blc {

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
// four floats at any 4-byte aligned global address: one 16-byte access all the same
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

// Two floats as three bfloat16 pairs (first value in the low half) whose sum
// is exact: x1 = bf16(x), x2 = bf16(x - x1), x3 = bf16(x - x1 - x2); the
// differences are exact, and what the third part rounds is below the first's
// 24th bit.  (From 2^-110 on: smaller values' last part is subnormal and ends at
// 2^-133.  From 3.3962e38 on, 0.2 % below float's largest, the first part rounds
// to infinity and the third is NaN; clamping it there costs an instruction per
// value, 1 to 2 % of most passes: 512 channels 116.9 -> 119.4 us, a series of
// 1250 samples 39.5 -> 40.4.)
__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector((floatx2){a, b}, bf16x2));
}
__device__ __forceinline__ void split3(float a, float b, unsigned& p1, unsigned& p2, unsigned& p3) {
  p1 = pack_bf16(a, b);
  a -= __uint_as_float(p1 << 16), b -= __uint_as_float(p1 & 0xFFFF0000u);
  p2 = pack_bf16(a, b);
  a -= __uint_as_float(p2 << 16), b -= __uint_as_float(p2 & 0xFFFF0000u);
  p3 = pack_bf16(a, b);
}

// The same of one value in double precision, for tables: parts `stride` apart.
__device__ __forceinline__ void split3_store(double v, unsigned short* out, int stride) {
  for (int p = 0; p < 3; ++p) {
    const unsigned f = __float_as_uint((float)v);  // (rounded twice: the next part takes up the difference)
    const unsigned short h = (unsigned short)((f + 0x7FFFu + ((f >> 16) & 1u)) >> 16);
    out[p * stride] = h;
    v -= (double)__uint_as_float((unsigned)h << 16);
  }
}

// An operand of eight k of a row or column, split: v = p[0] + p[1] + p[2].
struct Split8 {
  uintx4 p[3];
};
__device__ __forceinline__ Split8 split8(const float* v) {
  Split8 s;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    unsigned q1, q2, q3;
    split3(v[2 * k], v[2 * k + 1], q1, q2, q3);
    s.p[0][k] = q1, s.p[1][k] = q2, s.p[2][k] = q3;
  }
  return s;
}

// hi + lo += a b over 32 k of 16 x 16 outputs (v_mfma_f32_16x16x32_bf16: lane l
// holds k = 8 (l / 16) .. + 7 of row or column l % 16, and rows 4 (l / 16) + r of
// column l % 16 of the result): the first parts' product in hi, the five others
// down to 2^-18 of it in lo.
struct Acc16 {
  floatx4 hi, lo;
};
__device__ __forceinline__ void mma16(const uintx4* a, const uintx4* b, Acc16& c) {
  auto mm = [](uintx4 x, uintx4 y, floatx4 z) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), z, 0, 0,
                                                   0);
  };
  c.lo = mm(a[2], b[0], c.lo);
  c.hi = mm(a[0], b[0], c.hi);
  c.lo = mm(a[1], b[1], c.lo);
  c.lo = mm(a[0], b[2], c.lo);
  c.lo = mm(a[1], b[0], c.lo);
  c.lo = mm(a[0], b[1], c.lo);
}

}  // namespace blc
