// Six signed 8-bit digits of a scaled double (the operand format of gemm_i8s.h), without 64-bit conversions or shifts:
// adding 1.5 * 2^52 rounds the scaled value (|n| <= 2^46) to an integer in the low bits of the sum, half to even; 128 added to
// each of the five low bytes makes the borrows of signed digits, and flipping their top bits makes the bytes signed.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gptaq {

// exponent of the row scale: max < 2^e (the clamp keeps 2^(46 - e) a double; it is below anything fp32 inputs lead to)
__device__ __forceinline__ int digit_exponent(double mx) {
  return mx > 0.0 ? max(__builtin_amdgcn_frexp_exp(mx), -970) : 0;
}
__device__ __forceinline__ double digit_scale(int e) { return __builtin_bit_cast(double, (uint64_t)(1023 + 46 - e) << 52); }
__device__ __forceinline__ uint64_t digits_of(double v, double scale) {
  const double t = fma(v, scale, 6755399441055744.0);
  return (__builtin_bit_cast(uint64_t, t) + 0x8080808080ull) ^ 0x8080808080ull;
}
// w[i]: digit i (0: the most significant) of four values, the first in the lowest byte
__device__ __forceinline__ void pack_digits(uint64_t a, uint64_t b, uint64_t c, uint64_t d, uint32_t (&w)[6]) {
  const uint32_t al = (uint32_t)a, bl = (uint32_t)b, cl = (uint32_t)c, dl = (uint32_t)d;
  const uint32_t ah = (uint32_t)(a >> 32), bh = (uint32_t)(b >> 32), ch = (uint32_t)(c >> 32), dh = (uint32_t)(d >> 32);
  const uint32_t ab01 = __builtin_amdgcn_perm(bl, al, 0x05010400u), ab23 = __builtin_amdgcn_perm(bl, al, 0x07030602u);
  const uint32_t cd01 = __builtin_amdgcn_perm(dl, cl, 0x05010400u), cd23 = __builtin_amdgcn_perm(dl, cl, 0x07030602u);
  const uint32_t ab45 = __builtin_amdgcn_perm(bh, ah, 0x05010400u), cd45 = __builtin_amdgcn_perm(dh, ch, 0x05010400u);
  w[5] = __builtin_amdgcn_perm(cd01, ab01, 0x05040100u);
  w[4] = __builtin_amdgcn_perm(cd01, ab01, 0x07060302u);
  w[3] = __builtin_amdgcn_perm(cd23, ab23, 0x05040100u);
  w[2] = __builtin_amdgcn_perm(cd23, ab23, 0x07060302u);
  w[1] = __builtin_amdgcn_perm(cd45, ab45, 0x05040100u);
  w[0] = __builtin_amdgcn_perm(cd45, ab45, 0x07060302u);
}

}  // namespace gptaq
