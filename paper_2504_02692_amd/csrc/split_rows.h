// bf16 hi/lo split of the strictly upper triangle of an fp32 matrix, dXXT as the left operand of Theorem 4.2's first product (prepare.hip),
// made beside the first block of the factor sweep (factor_sweep.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gptaq {

__device__ __forceinline__ uint16_t bf16_rne(float f) {
  __bf16 b = (__bf16)f;
  return __builtin_bit_cast(uint16_t, b);
}
__device__ __forceinline__ float bf16_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// The two products of Theorem 4.2 only read the operand blocks of kSplitBlock^2 on and above the diagonal (their tiles start
// and their k ranges begin at multiples of a tile edge that divides it), so the others are not written: a third of
// extract_U_kernel's bytes and two thirds of split_rows's.
constexpr int kSplitBlock = 256;
// The operands are k-tile-major: a tile's rows of 32 k are one run, not 64 bytes of every row (whose stride is a power of two at
// n = 4096): 147 -> 118 us per product at n = 4096, 1.32 -> 1.10 ms at n = 11008.
__device__ __forceinline__ int64_t operand_at(int64_t row, int64_t k, int64_t np) { return (k >> 5) * np * 32 + row * 32 + (k & 31); }

// Rows flagged in `zero_rows` count as 0; padded to np x np; entries on and below the diagonal come out as 0, whatever they are: Eq. 17
// masks dXXT L to its strictly upper part and L is lower triangular, so entry (i, k) of dXXT only ever meets a non-zero of L when k > i.
// `info` (may be NULL): a NaN or Inf among the entries read is reported as info[0] = -(1 + row of the entry).
struct SplitRows { const float* A; int64_t lda; int n; const uint8_t* zero_rows; uint16_t *Ah, *Al; int64_t np; int32_t* info; };
// Columns cx * 256 .. + 255 of 32 rows, one workgroup of 256; ceil(np / 256) times np / 32 of them.  Eight columns of a row per thread and
// four rows in turn: a wavefront reads 128 bytes of each of 16 rows and writes 1 KB runs of a k-tile.  Bound by memory: as a launch
// of its own 17 us at n = 4096, 90 at 11008 (a column of four rows per thread: 23 and 129); rows that are not 16-byte aligned are read entry
// by entry.
constexpr int kSplitRowsPerWg = 32;
__device__ __forceinline__ void split_rows(const SplitRows& a, int64_t cx, int64_t ry) {
  typedef __attribute__((ext_vector_type(4))) float f4;
  typedef __attribute__((ext_vector_type(4))) uint32_t u4;
  const int t = threadIdx.x, lane = t & 63;
  const int64_t r0 = kSplitRowsPerWg * ry + (lane >> 2), c0 = cx * 256 + 64 * (t >> 6) + 8 * (lane & 3);
  if (cx * 256 / kSplitBlock < kSplitRowsPerWg * ry / kSplitBlock) return;
  const bool wide = ((uintptr_t)a.A & 15) == 0 && a.lda % 4 == 0;
  float v[4][8];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t r = r0 + 16 * (i & 1), c = c0 + 32 * (i >> 1);
    const float* src = a.A + (r < a.n ? r : a.n - 1) * a.lda;
    if (wide && c + 8 <= a.n) {
      const f4 x = *reinterpret_cast<const f4*>(src + c), y = *reinterpret_cast<const f4*>(src + c + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) { v[i][e] = x[e]; v[i][4 + e] = y[e]; }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[i][e] = src[c + e < a.n ? c + e : a.n - 1];
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t r = r0 + 16 * (i & 1), c = c0 + 32 * (i >> 1);
    if (c >= a.np || r >= a.np) continue;
    const bool none = r >= a.n || (a.zero_rows && a.zero_rows[r]);
    uint32_t h[8], l[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float x = !none && c + e < a.n && c + e > r ? v[i][e] : 0.f;
      if (a.info && !__builtin_isfinite(x)) atomicMin(a.info, -(1 + (int)r));
      h[e] = bf16_rne(x);
      l[e] = bf16_rne(x - bf16_f32((uint16_t)h[e]));
    }
    const int64_t o = operand_at(r, c, a.np);
    *reinterpret_cast<u4*>(a.Ah + o) = u4{h[0] | h[1] << 16, h[2] | h[3] << 16, h[4] | h[5] << 16, h[6] | h[7] << 16};
    *reinterpret_cast<u4*>(a.Al + o) = u4{l[0] | l[1] << 16, l[2] | l[3] << 16, l[4] | l[5] << 16, l[6] | l[7] << 16};
  }
}

}  // namespace gptaq
