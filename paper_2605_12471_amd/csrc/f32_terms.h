// fp32 operands as sums of three bf16 terms, for the fp32 attention kernels (attn_f32.hip says why and what it costs).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kvfold {

typedef __attribute__((ext_vector_type(16))) float floatx16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) unsigned uintx4;

constexpr int kTerms = 3;
// What the terms can hold: magnitudes below 2^60 (and a softmax scale below 2^20).  The products of a row's terms then stay
// below 2^127 and no partial sum overflows that the fp32 instructions' own sum would not; above, terms of opposite sign could
// meet as inf - inf where the product is infinite and the weight 0.  A sum of values times kProbe stays finite
// exactly if none of them reaches 2^60 (several that come within a factor of 128 may pass for one that does).
constexpr float kLargest = 0x1p60f, kProbe = 0x1p68f, kMaxScale = 0x1p20f;
// Values are split 2^23 times as large, so that their last bit, 2^-149 at the least, lies in the range of bf16; the sums of
// weights (at most 2^8) times values stay below 2^(8 + 83 + 24).  Queries and keys need no such factor: what a tiny one of
// them loses, at most 2^-126, moves a logit by less than 2^-38.  Nor do weights: one below 2^-103 loses at most
// 2^-126 of a sum of weights that is at least 1 (below 2^-126 it is 0).
constexpr float kValueScale = 0x1p23f, kValueUnscale = 0x1p-23f;
// Two values, as pair j of a fragment of eight of each term.
__device__ __forceinline__ void split2(float a, float b, uintx4 (&t)[kTerms], int j) {
#pragma unroll
  for (int i = 0; i < kTerms; ++i) {
    bf16x2 h;
    h[0] = (__bf16)a;
    h[1] = (__bf16)b;
    unsigned h2 = __builtin_bit_cast(unsigned, h);
    asm("" : "+v"(h2));  // (else the compiler converts each value once more for itself, where it is taken off)
    t[i][j] = h2;
    if (i + 1 < kTerms) {
      a -= __uint_as_float(h2 << 16);
      b -= __uint_as_float(h2 & 0xffff0000u);
    }
  }
}
// Eight values as three fragments of bf16 terms, each rounded to nearest, so that the second is at most 2^-8 and the third at
// most 2^-17 of the value.  (A value that is not finite leaves NaN in the lower terms.)
__device__ __forceinline__ void split8(const float (&x)[8], uintx4 (&t)[kTerms]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) split2(x[2 * j], x[2 * j + 1], t, j);
}
__device__ __forceinline__ floatx16 mfma16(const uintx4& a, const uintx4& b, const floatx16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

}  // namespace kvfold
