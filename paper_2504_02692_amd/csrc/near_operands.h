// The super-block kernel's operands of U and P (quantize_sb.hip), made in launches of their own or in a layer's first one (quantize.hip).
#pragma once
#include "common.h"

namespace gptaq {

constexpr int kSub = 16;                       // columns per sub-block
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

__device__ __forceinline__ uint16_t sb_bf16_rne(float f) {
  __bf16 b = (__bf16)f;
  return __builtin_bit_cast(uint16_t, b);
}
__device__ __forceinline__ float sb_bf16_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// What the super-block kernel reads of U and P, for super-block first + i (rows and columns sb0 = 1024 (first + i) on) and its sub-blocks e:
//   * left operands of the updates: for super-block column c behind the sub-block, the 16 entries S[sb0 + 16 e + k][sb0 + c], k = 0..15,
//     split into bf16 hi and lo, at ((64 i + e) * 1024 + c) * 16 + k of its array: the 32 columns x 16 k a wavefront needs for one MFMA
//     operand are 1 KB in a row (zeros for the sub-block's own columns, which take no update from it);
//   * the diagonal piece, 512 floats at diag + 512 (64 i + e): entry (step j, column c) of U at sb_diag_at(c, j) and of P 256 further on
//     (c > j; zeros outside the matrix), and 1 / U_jj at 256 + j (column 0 of P has no entry of its own).
// Workgroups of 256: tile = of 64 columns (kNearTiles), e = sub-block (kNearEvents), z = 2 i + (0 for U, 1 for P).
__host__ __device__ constexpr int sb_diag_at(int c, int j) { return 16 * c + 4 * ((j >> 2) ^ ((c >> 2) & 3)) + (j & 3); }   // (no bank conflicts)
constexpr int kNearTiles = kSbCols / 64, kNearEvents = kSbCols / kSub;
__device__ __forceinline__ void near_operands(const float* U, const float* P, int64_t ldh, int n, int first, const SbNear& o, int tile, int e, int z,
                                              float (&t)[kSub][65]) {
  const int c0 = tile * 64, isP = z & 1, place = z >> 1, sb0 = (first + place) * kSbCols;
  if (c0 + 64 <= kSub * e || sb0 + kSub * e >= n) return;  // entirely left of the sub-block, or no sub-block: never read
  const float* S = isP ? P : U;
  const int64_t ev = (int64_t)place * (kSbCols / kSub) + e;
  const int c = threadIdx.x & 63, kq = threadIdx.x >> 6;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int k = kq + 4 * p;
    const int64_t row = (int64_t)sb0 + kSub * e + k, col = (int64_t)sb0 + c0 + c;
    t[k][c] = (row < n && col < n) ? S[row * ldh + col] : 0.f;
  }
  __syncthreads();
  const int own = kSub * e - c0;                           // the sub-block's own columns, from the tile's first
  if (own >= 0) {
    const int j = threadIdx.x & 15, cc = threadIdx.x >> 4;
    const float v = t[j][own + cc];
    float* d = o.diag + 512 * ev;
    if (!isP) {
      d[sb_diag_at(cc, j)] = cc > j ? v : 0.f;
      if (cc == j) d[256 + j] = v != 0.f ? 1.f / v : 0.f;
    } else if (cc > 0) {
      d[256 + sb_diag_at(cc, j)] = cc > j ? v : 0.f;
    }
  }
  const int cc = threadIdx.x >> 2, k4 = (threadIdx.x & 3) * 4;
  uint16_t h[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float v = cc >= own + kSub ? t[k4 + i][cc] : 0.f;
    h[i] = sb_bf16_rne(v);
    l[i] = sb_bf16_rne(v - sb_bf16_f32(h[i]));
  }
  const int64_t at = (ev * kSbCols + c0 + cc) * kSub + k4;
  u32x2 vh = {(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16)};
  u32x2 vl = {(uint32_t)l[0] | ((uint32_t)l[1] << 16), (uint32_t)l[2] | ((uint32_t)l[3] << 16)};
  *reinterpret_cast<u32x2*>(o.left + 2 * isP * o.stride + at) = vh;
  *reinterpret_cast<u32x2*>(o.left + (2 * isP + 1) * o.stride + at) = vl;
}

}  // namespace gptaq
