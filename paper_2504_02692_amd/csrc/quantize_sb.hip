// Algorithm 1, lines 5-13 for one super-block of up to 1024 columns in a single launch.
//
// Rows of W never interact (Step 1: all output channels are solved in parallel with one shared
// factor), so a workgroup owns 64 rows for the whole super-block and needs no grid-level
// synchronisation: the 64 x 1024 slice of W lives in the accumulator registers of its eight
// wavefronts from the first column of the super-block to the last, and every update of
// Eq. 15 / Eq. 18 that stays inside the super-block is applied there.
//
// Three levels of lazy batching (a re-association of the sums of Eq. 18, which leaves the result
// independent of the blocking):
//   * 16 columns ("sub-block"): the sequential column steps of lines 7-10, one row per lane, fp32
//     FMAs, the 16 x 16 diagonal pieces of U and P in registers, broadcast by DPP;
//   * the rest of the super-block: after each sub-block, W[:, later] += [-E | V] [U; P][sub-block, later]
//     on the matrix cores (bf16 hi/lo split of both sides, three products per term), straight into
//     the accumulators that hold W;
//   * the columns after the super-block: one GEMM per super-block, outside this kernel, from the
//     -E and V this kernel leaves behind in the GEMM's operand format.
//
// Who holds what.  The super-block is eight blocks of 128 columns and wave w of the workgroup's eight holds block w, as
// four 32-column pieces of two 32 x 32 MFMA accumulator tiles (rows 0-31 and 32-63) of the TRANSPOSED
// product  W^T += [U; P]^T [-E | V]^T :  lane l, register v of a tile holds row l % 32 of the tile,
// column 8 (v / 4) + 4 (l / 32) + v % 4 of the piece.  v_permlane32_swap of the registers of the two
// tiles turns that into "one row per lane" for the sequential steps, and turns -E and V of a sub-block back into
// MFMA operands without a trip through LDS.
//
// A wave's life has three parts.  Updater: its block lies after the one being worked on; it applies every sub-block's
// update to its four pieces, the left operands fetched into registers a sub-block ahead.  Owner: it runs the column
// steps of its eight sub-blocks; of its own block it updates the piece that its next sub-block lies in at once, the other pieces beside
// that sub-block's column steps.  Finished.  One workgroup barrier per sub-block publishes its -E and V.  What the owner needs
// next from memory (diagonal pieces of U and P, left operands) the others fetch into LDS, and they form and store its results.
//
// What bounds it: the owner's chain, of the 64 sub-blocks about 4.3K clocks each in the first four blocks, where an updater shares the owner's
// SIMD, and 3.7K in the last four: 1.9K of column steps (376 vector instructions at 5 clocks; 650 more when 24 MFMAs run beside them),
// 200 to bring the 16 columns into one row per lane, 1.0K for the operands and the 12 MFMAs of the next sub-block's piece; and 3.7K from
// one block to the next (48 MFMAs of the new owner, the group's range and grid).  The matrix pipes of a SIMD with two updaters need 3.1K
// a sub-block.
// What that took, on the way from 5.3K a sub-block (151 -> 137 us for 1024 columns of 4096 rows, 64 workgroups, with nothing beside it;
// rows' outputs the same bits): W^ and codes formed by the wavefront that stores them; V split and LDS written under the next
// piece's MFMAs; single MFMAs between column steps (7 clocks of the wavefront each, but 32 behind another MFMA); loads to LDS shared out
// over all wavefronts and hidden from the compiler's wait counts; updaters' loads one by one between their MFMAs and a whole
// sub-block ahead.
#include "common.h"
#include "near_operands.h"
#include <utility>

namespace gptaq {

constexpr int kSbBlocks = kSbCols / 128;       // 128-column blocks per super-block

// Uniform affine min-max grid with 0 inside the range; the few operations per group are done in fp64 so
// that the fp32 scale is the correctly rounded (xmax - xmin) / maxq.
__device__ __forceinline__ double sb_grid_params(float xmin, float xmax, float maxq, int sym, float& scale, float& zero) {
  double lo = fmin((double)xmin, 0.0), hi = fmax((double)xmax, 0.0);
  if (sym) { hi = fmax(fabs(lo), hi); lo = -hi; }
  if (lo == 0.0 && hi == 0.0) { lo = -1.0; hi = 1.0; }
  const double base = (hi - lo) / (double)maxq;
  scale = (float)base;
  zero = sym ? (maxq + 1.f) * 0.5f : (float)rint(-lo / (double)scale);
  return base;
}
// scale of candidate i of the clip-range search
__device__ __forceinline__ float sb_clip_scale(double base, int i, int grid) {
  return (float)((1.0 - (double)i / (double)grid) * base);
}

__global__ __launch_bounds__(256) void near_operands_kernel(const float* U, const float* P, int64_t ldh, int n, int first, SbNear o) {
  __shared__ float t[kSub][65];
  near_operands(U, P, ldh, n, first, o, blockIdx.x, blockIdx.y, blockIdx.z, t);
}

// ---------------------------------------------------------------------------------------------------
constexpr int kSbWaves = 8;                      // one 128-column block each
constexpr int kSbRowLd = 20;                     // padded row of 16 results in LDS, in floats
static_assert(kSbBlocks == kSbWaves, "one block per wave");
struct SbShared {
  // operands [-E | V]^T of a sub-block's update in MFMA fragment order: [buffer][-E hi, -E lo, V hi, V lo][row half][lane]
  u32x4 frag[2][4][2][64];
  // left operands for the owner's own pieces: [buffer][piece][U hi, U lo, P hi, P lo], 1 KB each
  u32x4 left[4][4][4][64];
  float d[2][64][kSbRowLd];                      // W^ of a sub-block in steps of the grid, less the zero-point, a row per row
  float grid[2][64][2];                          // scale and zero-point of each row
  float diag[4][2 * kSub * kSub];                // diagonal pieces of U and P and 1 / U_jj (see near_operands_kernel)
};

// Clip-range search of a group of the current weights (Section 5.1; candidates p = 1 - i / grid of the min-max range, the smallest
// sum of squared errors wins, the earlier one on ties).  The owner stages the group's weights, one row per lane, and all eight
// wavefronts search: each takes every eighth candidate, so no sum crosses lanes.  Bound by its five instructions per weight and
// candidate: ~17 us per 128 columns and 80 candidates of 64 rows, whatever the number of workgroups.  (With one row per wavefront,
// two columns per lane and a reduction over the lanes for each candidate, in a launch per 128 columns, a 4096 x 4096 layer took
// 3.92 ms; 1.57.)
// A sum is a tree over the columns: its error against 64 bits is 4.2e-8 rms, 1.8e-7 at most (20000 groups of 16, 32, 64 or 128 normal
// weights; one chain of 128 FMAs: 1.7e-7 and 8.8e-7, the reduction over the lanes 4.3e-8 and 1.9e-7).
// A wavefront sums five candidates at a time, then two, then one, so that the time follows their number: 64 x 1024 in groups of 128
// with 1 / 8 / 40 / 80 / 100 / 160 candidates 184 / 189 / 246 / 323 / 361 / 475 us.  (Ten at a time, the last ones repeated to fill
// them up: 281 / 316 / 316 / 316 / 471 / 471, and 128 columns with up to 20 candidates took 1.2 to 1.4 times as long as one launch per
// 128 columns did.)
struct SbClip {
  float w[128][64];                              // [column of the group][row]
  double base[64];                               // full scale of the row's group, not yet rounded
  float zero[64];
  float err[kSbWaves][64];                       // the best of a wavefront's candidates
  int cand[kSbWaves][64];
};

__device__ __forceinline__ uint32_t sb_lds_address(const void* p) { return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p; }

// 1 KB per wavefront from global memory straight into LDS: lane l's 16 bytes land at lds + 16 l (lds the same in all lanes).
// It writes no register.  In asm because the compiler, once it has seen such a load, waits for all of a wavefront's loads before each
// of its own reads of LDS and before each use of a loaded register, and an updater stood for a memory latency in every sub-block.  Unseen,
// it can only make the compiler's waits for loads longer (they count in order); the waits for it are written out before a barrier.
__device__ __forceinline__ void sb_load_lds(const void* src, void* lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               : : "s"(__builtin_amdgcn_readfirstlane(sb_lds_address(lds))), "v"(src) : "memory", "m0");
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for every outstanding global
// store (the results a wave has just written, which nobody in this kernel reads back): a microsecond per
// sub-block.
__device__ __forceinline__ void sb_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// w += (lane C of each group of 16 lanes of s) * e: the 16 entries of a row of U (or P) sit in the 16 lanes of s, so a
// column step needs neither LDS reads nor a register per entry.  s must not have been written by the two instructions
// before (the compiler does not look into the asm): see sb_pin; tests/test_dpp_hazards.py checks the machine code for it.
template <int C> __device__ __forceinline__ void sb_fmac_lane(float& w, float s, float e) {
  asm("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(w) : "v"(s), "v"(e), "n"(C));
}
template <int C> __device__ __forceinline__ float sb_mul_lane(float s, float e) {
  float r;
  asm("v_mul_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(s), "v"(e), "n"(C));
  return r;
}
__device__ __forceinline__ void sb_pin(float (&s)[kSub]) {
  asm volatile("s_nop 1" : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]), "+v"(s[3]), "+v"(s[4]), "+v"(s[5]), "+v"(s[6]), "+v"(s[7]),
               "+v"(s[8]), "+v"(s[9]), "+v"(s[10]), "+v"(s[11]), "+v"(s[12]), "+v"(s[13]), "+v"(s[14]), "+v"(s[15]));
}

// two fp32 -> bf16 pair (round to nearest even) and what the rounding left over
__device__ __forceinline__ u32x2 sb_split2(float a, float b) {
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  const uint32_t hi = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
  const float ra = a - __uint_as_float(hi << 16), rb = b - __uint_as_float(hi & 0xffff0000u);
  return u32x2{hi, __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{ra, rb}), bf16x2))};
}

// -E of columns J - 1 and J, e = t / U_jj rounded to fp32, as bf16 hi and lo: lo carries what hi leaves of the product before that
// rounding (one FMA), as far as 8 bits go.  (Three instructions per two columns more than the residual of the rounded e1, which
// moved half of the later groups' scales by their last bit: 1024 columns 152.3 -> 153.9 us.)
template <int J>
__device__ __forceinline__ u32x2 sb_split_e(float e0, float e1, float t0, float t1, float dreg) {
  const uint32_t hi = sb_split2(e0, e1)[0], neg = hi ^ 0x80008000u;
  float r0 = __uint_as_float(neg << 16), r1 = __uint_as_float(neg & 0xffff0000u);
  sb_fmac_lane<J - 1>(r0, dreg, t0);
  sb_fmac_lane<J>(r1, dreg, t1);
  return u32x2{hi, sb_split2(r0, r1)[0]};
}

// registers 8 HALF .. 8 HALF + 7 of a piece's two tiles -> the 16 columns of the sub-block, one row per lane
template <int HALF>
__device__ __forceinline__ void sb_extract(const f32x16 (&t)[2], float (&w)[kSub]) {
#pragma unroll
  for (int vv = 0; vv < 8; ++vv) {
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(t[0][8 * HALF + vv]), __float_as_uint(t[1][8 * HALF + vv]),
                                                     false, false);
    const int c = 8 * (vv >> 2) + (vv & 3);
    w[c] = __uint_as_float(r[0]);          // lanes 0-31: tile 0, lanes 32-63: tile 1, columns of lane half 0
    w[c + 4] = __uint_as_float(r[1]);      // the columns lane half 1 held
  }
}

// t += left operands (U hi, U lo, P hi, P lo of 32 columns) x fragments (-E hi, -E lo, V hi, V lo): three products per term.
// between(m) comes behind the m-th MFMA.
template <class Between>
__device__ __forceinline__ void sb_piece_update(f32x16 (&t)[2], const u32x4 (&left)[4], const u32x4 (&fr)[4][2], bool useE, bool useP,
                                                Between&& between) {
  int m = 0;
#pragma unroll
  for (int tm = 0; tm < 2; ++tm) {
    if (!(tm ? useP : useE)) continue;
    const bf16x8 ah = __builtin_bit_cast(bf16x8, left[2 * tm]), al = __builtin_bit_cast(bf16x8, left[2 * tm + 1]);
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int rh = 0; rh < 2; ++rh) {
        t[rh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q == 2 ? al : ah, __builtin_bit_cast(bf16x8, fr[2 * tm + (q == 1)][rh]), t[rh], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        between(m++);
        __builtin_amdgcn_sched_barrier(0);
      }
  }
}

// The grid of a row whose range is [lo, hi] (the lanes of a row agree), its reciprocal, and its place in the outputs.
struct SbGrid { float sc, zr, isc; };

// w[J + 1 ..] += (a row of U or P, from its column J + 1 on) * e
template <int J, int... C>
__device__ __forceinline__ void sb_row_update(float (&w)[kSub], float s, float e, std::integer_sequence<int, C...>) {
  (sb_fmac_lane<J + 1 + C>(w[J + 1 + C], s, e), ...);
}

// One column step (lines 7-10 of Algorithm 1), one row per lane, and those after it.  w[J] stays the value before rounding, d[J] is
// its rounded value in steps of the grid, less the zero-point.  between(2 J) and between(2 J + 1) put other work of the wavefront
// beside step J.
template <int TERMS, int J, class Between>
__device__ __forceinline__ void sb_steps(float (&w)[kSub], float (&d)[kSub], const float (&u)[kSub], const float (&p)[kSub], float dreg,
                                         const SbGrid& g, float dlo, float dhi, float e_prev, float t_prev, u32x4 (&pe)[2][2],
                                         Between&& between) {
  if constexpr (J < kSub) {
    between(std::integral_constant<int, 2 * J>{});
    const float v = w[J];
    // code - zero = clamp(rint(v / scale), -zero, maxq - zero): the same integers as clamp(rint(.) + zero, 0, maxq)
    // - zero, with a shorter dependency chain in front of the updates (one median instead of add, max, min, sub)
    d[J] = __builtin_amdgcn_fmed3f(rintf(v * g.isc), dlo, dhi);
    const float t = fmaf(g.sc, d[J], -v);                  // W^ - v, rounded once
    const float e1 = sb_mul_lane<J>(dreg, t);              // -E_J
    constexpr std::make_integer_sequence<int, kSub - 1 - J> later{};
    if constexpr (TERMS & 2) sb_row_update<J>(w, p[J], v, later);
    between(std::integral_constant<int, 2 * J + 1>{});
    if constexpr (TERMS & 1) sb_row_update<J>(w, u[J], e1, later);
    if constexpr (J & 1) {
      const u32x2 x = sb_split_e<J>(e_prev, e1, t_prev, t, dreg);
      pe[0][J >> 3][(J >> 1) & 3] = x[0];
      pe[1][J >> 3][(J >> 1) & 3] = x[1];
    }
    sb_steps<TERMS, J + 1>(w, d, u, p, dreg, g, dlo, dhi, e1, t, pe, between);
  }
}

// one row and two chunks of eight columns per lane -> one chunk and a row of each half per lane (an MFMA operand)
__device__ __forceinline__ void sb_to_operand(u32x4 (&x)[2]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const u32x2 r = __builtin_amdgcn_permlane32_swap(x[0][k], x[1][k], false, false);
    x[0][k] = r[0];
    x[1][k] = r[1];
  }
}

// Of an owner's update by its sub-block `eb` of the block: the piece its next sub-block lies in is updated at once, and pieces
// first_deferred(eb) .. 3 beside the next sub-block's column steps.  (A group of 64 may start at sub-block 4 and needs every piece from 2
// on; more than two pieces would not fit beside the steps.)
__host__ __device__ constexpr int sb_next_piece(int eb) { return (eb + 1) >> 1; }
__host__ __device__ constexpr int sb_first_deferred(int eb) { return eb < 0 || eb == 3 ? 4 : eb == 0 ? 2 : sb_next_piece(eb) + 1; }

// FAST: rows of W and of the codes are 16-byte aligned and n is a multiple of 16 (vector loads and stores).
// TERMS: the update terms of Eq. 15 that are applied (3: both; a run-time choice would cost branches around every MFMA group,
// and with them spills).
// CLIP: the range of every group is searched (groups only; per-channel ranges come with the call).
template <bool FAST, int TERMS, bool CLIP>
__global__ __launch_bounds__(64 * kSbWaves) void quant_sb_kernel(SbArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char sb_smem[];
  SbShared& sh = *reinterpret_cast<SbShared*>(sb_smem);
  SbClip& cl = *reinterpret_cast<SbClip*>(sb_smem + sizeof(SbShared));      // (with CLIP only)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, lh = lane >> 5;
  const int row0 = blockIdx.x * 64;
  const int sbw = a.sbw;                                  // columns of this super-block
  const int nev = (sbw + kSub - 1) / kSub;
  constexpr bool useE = TERMS & 1, useP = TERMS & 2, update = TERMS != 0;
  const uint32_t lane_off = (uint32_t)(l32 * kSub + 8 * lh);       // this lane's 16 bytes of 32 columns x 16 k of a left operand
  const int first_own = min(8 * wave, nev), last_own = min(8 * wave + 8, nev);

  // ---- W -> accumulators.  Out-of-range elements read a clamped (valid) address and are replaced by 0,
  // so the loads need no branches.  Dead inputs were zeroed in W before this kernel.
  f32x16 acc[4][2];
  if (first_own < last_own) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int rh = 0; rh < 2; ++rh) {
        const int row = row0 + 32 * rh + l32;
        const float* src = a.W + (int64_t)min(row, a.m - 1) * a.ldw + a.sb0;
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
          const int c = 128 * wave + 32 * i + 8 * vq + 4 * lh;    // super-block column of element 0
          if (FAST) {
            const bool ok = row < a.m && c < sbw;
            const f32x4 x = *reinterpret_cast<const f32x4*>(src + min(c, sbw - 4));
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[i][rh][4 * vq + q] = ok ? x[q] : 0.f;
          } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float x = src[min(c + q, sbw - 1)];
              acc[i][rh][4 * vq + q] = (row < a.m && c + q < sbw) ? x : 0.f;
            }
          }
        }
      }
    }
  }

  // ---- what the wavefronts that do not own block b do for the one that does.
  // All: fetch what it needs besides its accumulators, the diagonal pieces of U and P and the left operands of the update of its own
  // later columns, both into buffer x & 3 and two sub-blocks ahead (the owner reads the diagonal pieces of x before barrier x - 1, and the
  // last left operands of x before barrier x + 1).  The loads are requested behind a barrier and waited for in front of the next one.
  // (A wavefront hands one such load over in some 80 clocks.  Up to 18 of them in one wavefront made it late at the barrier
  // while it was an updater itself, in the first two blocks: 3K clocks a sub-block.)
  // And store its results: wave b - 1, or all for the first block.
  auto own_lane = [&]() {                                 // (the search leaves no registers for addresses kept between the events)
    int l = lane;
    asm volatile("" : "+v"(l));
    return l;
  };
  auto request = [&](int x, int t) {                        // item t of sub-block x
    const int lane = own_lane();
    const int eb = x & 7, count = update ? 4 * (4 - sb_next_piece(eb)) + 2 : 0;
    const int i = 3 - ((t - 2) >> 2), q = (t & 3) ^ 2;      // t = 0, 1: the diagonal pieces; then the four left operands of piece 3, 2, ...
    if (t >= count) return;
    if (t < 2) sb_load_lds(a.near.diag + 512 * x + 256 * t + 4 * lane, &sh.diag[x & 3][256 * t]);
    else if (q < 2 ? useE : useP)
      sb_load_lds(a.near.left + q * a.near.stride + ((x * kSbCols + 128 * (x >> 3) + 32 * i) * kSub + (lane & 31) * kSub + 8 * (lane >> 5)),
                  &sh.left[x & 3][i][q][0]);
  };
  // results of sub-block x, from LDS to memory.  W^ and codes (formed here: the owner has the longer chain), 16 rows at a time:
  auto store_rows = [&](int x, int it) {
    const int lane = own_lane();
    const int buf = x & 1, colg = a.sb0 + kSub * x;
    const int r = FAST ? 16 * it + (lane >> 2) : 16 * it + (lane & 15), c = FAST ? 4 * (lane & 3) : 4 * (lane >> 4);
    const f32x4 d = *reinterpret_cast<const f32x4*>(&sh.d[buf][r][c]);
    const float sc = sh.grid[buf][r][0], zr = sh.grid[buf][r][1];
    uint32_t cw = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) cw = __builtin_amdgcn_cvt_pk_u8_f32(d[k] + zr, k, cw);
    if (row0 + r >= a.m) return;
    float* w = a.W + (int64_t)(row0 + r) * a.ldw + colg + c;
    uint8_t* code = a.codes + (int64_t)(row0 + r) * a.n + colg + c;
    if (FAST) {
      *reinterpret_cast<f32x4*>(w) = f32x4{sc * d[0], sc * d[1], sc * d[2], sc * d[3]};
      *reinterpret_cast<uint32_t*>(code) = cw;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (colg + c + k < a.n) {
          w[k] = sc * d[k];
          code[k] = (uint8_t)(cw >> (8 * k));
        }
    }
  };
  // and, 32 rows at a time, -E hi, -E lo, V hi and V lo for the update of the columns after the super-block
  auto store_operands = [&](int x, int it) {
    const int lane = own_lane();
    const int item = lane + 64 * it, r = item >> 1, ch = item & 1;
    u32x4 v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = sh.frag[x & 1][q][r >> 5][32 * ch + (r & 31)];
    uint16_t* dst = a.EV + (int64_t)(x >> 1) * a.evkt + (int64_t)(row0 + r) * 32 + kSub * (x & 1) + 8 * ch;
    if (row0 + r >= a.m) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) *reinterpret_cast<u32x4*>(dst + q * a.evstride) = v[q];
  };
  // this wavefront's part in the time between barrier x - 1 and barrier x, begin and end (x == nev: after the last barrier)
  auto help_begin = [&](int x) {
    const int r = (wave - (x >> 3) - 1) & 7;               // (7: the owner)
    if (r < 7 && x + 2 < nev) {
#pragma unroll
      for (int k = 0; k < 3; ++k) request(x + 2, r + 7 * k);
    }
  };
  auto help_end = [&](int x) {
    // (in the first block no wavefront is without updates, and each takes a share)
    const int b = min(x, nev - 1) >> 3, r = b == 0 ? wave - 1 : wave == b - 1 ? 0 : -1, step = b == 0 ? 7 : 1;
    if (x < 1 || r < 0) return;
    for (int t = r; t < (a.EV ? 6 : 4); t += step) {
      if (t < 4) store_rows(x - 1, t);
      else store_operands(x - 1, t - 4);
    }
  };
  for (int k = 0; k < 3; ++k) {
    request(0, wave + 8 * k);
    if (nev > 1) request(1, wave + 8 * k);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // this wavefront's part of the search for the group that starts at sub-block x; all wavefronts come here at the same x
  auto search = [&]() __attribute__((always_inline)) {
    sb_barrier();
    const double base = cl.base[lane];
    const float dlo = -cl.zero[lane], dhi = a.maxq + dlo;
    float best = __builtin_inff();
    int cand = 0;
    // K candidates at a time, i, i + kSbWaves, ...: a weight is read from LDS once for all of them.  Four squares are one chain, the
    // chains of 16 columns are added in pairs, and these sums again, like the digits of a binary counter: held[l] is the sum of the
    // last 16 << l columns while it has no partner.
    auto offer = [&](auto count, int i) __attribute__((always_inline)) {
      constexpr int K = decltype(count)::value;
      float sc[K], isc[K], held[3][K], sum[K];
#pragma unroll
      for (int k = 0; k < K; ++k) {
        sc[k] = sb_clip_scale(base, i + k * kSbWaves, a.clip_grid);
        isc[k] = 1.f / sc[k];
      }
      // (the next four weights are requested before the squares of these)
      float x[4], nx[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = cl.w[q][lane];
#pragma clang loop unroll(disable)
      for (int c = 0; c < a.group; c += kSub) {
        float half[K];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          const int cn = min(c + 4 * h + 4, a.group - 4);
#pragma unroll
          for (int q = 0; q < 4; ++q) nx[q] = cl.w[cn + q][lane];
          float e[K];
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int k = 0; k < K; ++k) {
              const float d = fmaf(sc[k], __builtin_amdgcn_fmed3f(rintf(x[q] * isc[k]), dlo, dhi), -x[q]);
              e[k] = q == 0 ? d * d : fmaf(d, d, e[k]);
            }
#pragma unroll
          for (int k = 0; k < K; ++k) {
            if (h == 0) sum[k] = e[k];
            if (h == 1) sum[k] += e[k];
            if (h == 2) half[k] = e[k];
            if (h == 3) sum[k] += half[k] + e[k];
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) x[q] = nx[q];
        }
        const int done = c / kSub + 1;                       // (1, 2, 4 or 8 in the end: then sum has every pair in it)
        if (done & 1) {
#pragma unroll
          for (int k = 0; k < K; ++k) held[0][k] = sum[k];
        } else {
#pragma unroll
          for (int k = 0; k < K; ++k) sum[k] += held[0][k];
          if (done & 2) {
#pragma unroll
            for (int k = 0; k < K; ++k) held[1][k] = sum[k];
          } else {
#pragma unroll
            for (int k = 0; k < K; ++k) sum[k] += held[1][k];
            if (done & 4) {
#pragma unroll
              for (int k = 0; k < K; ++k) held[2][k] = sum[k];
            } else {
#pragma unroll
              for (int k = 0; k < K; ++k) sum[k] += held[2][k];
            }
          }
        }
      }
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (sum[k] < best) { best = sum[k]; cand = i + k * kSbWaves; }
    };
    int i = wave;
    for (; i + 4 * kSbWaves < a.clip_steps; i += 5 * kSbWaves) offer(std::integral_constant<int, 5>{}, i);
    for (; i + kSbWaves < a.clip_steps; i += 2 * kSbWaves) offer(std::integral_constant<int, 2>{}, i);
    if (i < a.clip_steps) offer(std::integral_constant<int, 1>{}, i);
    cl.err[wave][lane] = best;
    cl.cand[wave][lane] = cand;
    sb_barrier();
  };
  auto group_starts = [&](int x) { return CLIP && ((kSub * (x & 7)) & (a.group - 1)) == 0; };      // (groups are powers of two here)

  // ================= updater: sub-blocks before this wave's own
  int e = 0;
  if (first_own < last_own && first_own > 0) {
    // left operands of the four pieces, a register set each.  A piece's set is filled again between the MFMAs of the piece behind it, a
    // load at a time, for the next sub-block.  (Two sets, filled two pieces ahead: an L2 round trip is longer than the MFMAs of a piece.
    // Four loads in a row behind each piece: up to 28 wavefront loads of all updaters at once, and the matrix cores idle.)
    constexpr int PER = 2 * ((TERMS & 1) + (TERMS >> 1));  // loads per piece
    u32x4 left[4][4];
    auto load_left = [&](int x, int i, int k) {            // the k-th of them
      const int q = useE ? k : k + 2;
      left[i][q] = *reinterpret_cast<const u32x4*>(a.near.left + q * a.near.stride + ((x * kSbCols + 128 * wave + 32 * i) * kSub + (int)lane_off));
    };
    auto load_first = [&](int x) {
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < PER; ++k) load_left(x, i, k);
    };
    help_begin(0);
    __builtin_amdgcn_sched_barrier(0);
    if (update) load_first(0);
    for (; e < first_own; ++e) {
      if (group_starts(e)) {
        search();
        if (update) load_first(e);                         // (again: the search leaves no registers for them)
      }
      // (the requests for the owner are older than those for this wavefront's next update)
      if (update) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(3 * PER) : "memory");
      help_end(e);
      sb_barrier();
      if (!update) continue;
      if (e == first_own - 1) __builtin_amdgcn_s_setprio(3);   // the other waves wait for this one from here on
      u32x4 fr[4][2];
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int rh = 0; rh < 2; ++rh) fr[q][rh] = sh.frag[e & 1][q][rh][lane];
      help_begin(e + 1);
      const int nx = min(e + 1, first_own - 1);            // (the last requests are repeats that nobody uses)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        sb_piece_update(acc[i], left[i], fr, useE, useP, [&](int m) {
          if (m % 3 == 2 && m / 3 < PER) load_left(i == 0 ? e : nx, (i + 3) & 3, m / 3);
        });
    }
  }

  // ================= owner: the column steps of this wave's eight sub-blocks
  if (first_own < last_own) {
    SbGrid g{1.f, 0.f, 1.f};
    const int row = row0 + lane;
    if (a.group <= 0) {
      if (row < a.m) { g.sc = a.scales[row]; g.zr = a.zeros[row]; }
      g.isc = 1.f / g.sc;
    }
    auto new_grid = [&](float lo, float hi, int x) __attribute__((always_inline)) {      // (with CLIP the group's weights have been staged)
      const double base = sb_grid_params(lo, hi, a.maxq, a.sym, g.sc, g.zr);
      if (CLIP) {
        cl.base[lane] = base;
        cl.zero[lane] = g.zr;
        search();
        float best = __builtin_inff();
        int cand = -1;
#pragma unroll
        for (int q = 0; q < kSbWaves; ++q) {
          const float err = cl.err[q][lane];
          const int i = cl.cand[q][lane];
          if (err < best || (err == best && i < cand)) { best = err; cand = i; }
        }
        if (cand >= 0) g.sc = sb_clip_scale(base, cand, a.clip_grid);
      }
      g.isc = 1.f / g.sc;
      if (row < a.m) {
        const int64_t o = (int64_t)row * a.G + ((a.sb0 + kSub * x) >> (31 - __builtin_clz(a.group)));
        a.scales[o] = g.sc;
        a.zeros[o] = g.zr;
      }
    };
    __builtin_amdgcn_s_setprio(3);
    float u[kSub], p[kSub], dreg;
    auto load_diag = [&](int x) {
      const int c = lane & 15;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 a4 = *reinterpret_cast<const f32x4*>(&sh.diag[x & 3][sb_diag_at(c, 4 * q)]);
        const f32x4 b4 = *reinterpret_cast<const f32x4*>(&sh.diag[x & 3][256 + sb_diag_at(c, 4 * q)]);
#pragma unroll
        for (int k = 0; k < 4; ++k) { u[4 * q + k] = a4[k]; p[4 * q + k] = b4[k]; }
      }
      dreg = sh.diag[x & 3][256 + c];
    };
    if (!CLIP) load_diag(first_own);
    auto event = [&](auto number) {
      constexpr int EB = decltype(number)::value;
      constexpr int R = EB >> 1, HALF = EB & 1, NEXT = sb_next_piece(EB);  // current piece, its half, the next sub-block's piece
      const int x = first_own + EB, buf = x & 1;
      if (x >= last_own) return;
      // ---- group range over the current (error-compensated) weights: the group's pieces are all in this wave
      if (HALF == 0 && a.group >= 32 && ((32 * R) & (a.group - 1)) == 0) {
        float lo[2] = {0.f, 0.f}, hi[2] = {0.f, 0.f}, mn[2], mx[2];
#pragma unroll
        for (int rh = 0; rh < 2; ++rh) {
#pragma unroll
          for (int i = R; i < 4; ++i)
            if (32 * (i - R) < a.group) {
#pragma unroll
              for (int v = 0; v < 16; ++v) { lo[rh] = fminf(lo[rh], acc[i][rh][v]); hi[rh] = fmaxf(hi[rh], acc[i][rh][v]); }
            }
          const u32x2 r0 = __builtin_amdgcn_permlane32_swap(__float_as_uint(lo[rh]), __float_as_uint(lo[rh]), false, false);
          const u32x2 r1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(hi[rh]), __float_as_uint(hi[rh]), false, false);
          mn[rh] = fminf(__uint_as_float(r0[0]), __uint_as_float(r0[1]));
          mx[rh] = fmaxf(__uint_as_float(r1[0]), __uint_as_float(r1[1]));
        }
        if (CLIP) {
#pragma unroll
          for (int i = R; i < 4; ++i)
            if (32 * (i - R) < a.group) {
#pragma unroll
              for (int rh = 0; rh < 2; ++rh)
#pragma unroll
                for (int v = 0; v < 16; ++v) cl.w[32 * (i - R) + 8 * (v >> 2) + 4 * lh + (v & 3)][32 * rh + l32] = acc[i][rh][v];
            }
        }
        new_grid(lh ? mn[1] : mn[0], lh ? mx[1] : mx[0], x);
      }
      float w[kSub], d[kSub];
      const bool late = CLIP && a.group == kSub;           // (a search in between leaves no registers for them)
      if (CLIP && !late) load_diag(x);                     // (without a search they have been read already)
      sb_extract<HALF>(acc[R], w);
      if (a.group == kSub) {                               // the group is this sub-block: its grid comes from the registers
        float mn = 0.f, mx = 0.f;
#pragma unroll
        for (int c = 0; c < kSub; ++c) {
          mn = fminf(mn, w[c]);
          mx = fmaxf(mx, w[c]);
          if (CLIP) cl.w[c][lane] = w[c];
        }
        new_grid(mn, mx, x);
      }
      if (late) load_diag(x);
      sb_pin(u);
      sb_pin(p);
      asm volatile("s_nop 1" : "+v"(dreg));
      // ---- the column steps.  Beside them, two MFMAs (one product for both row halves) per step from step 1 on: what the sub-block
      // before has left of its update.  Their operands are read from LDS one step ahead.  (An MFMA alone takes 7 clocks of the
      // wavefront's time here; right behind another one 32.)
      constexpr int D0 = sb_first_deferred(EB - 1), PER = update ? 3 * ((TERMS & 1) + (TERMS >> 1)) : 0, NSLOT = (4 - D0) * PER;
      static_assert(NSLOT < kSub, "a product per step");
      u32x4 dl[2], df[2][2];
      auto between = [&](auto point) {
        constexpr int J = decltype(point)::value / 2, rh = decltype(point)::value & 1;
        if constexpr (rh == 0 && J > 0 && J % 4 == 0)
          *reinterpret_cast<f32x4*>(&sh.d[buf][lane][J - 4]) = f32x4{d[J - 4], d[J - 3], d[J - 2], d[J - 1]};
        if constexpr (NSLOT > 0) {
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (J < NSLOT && rh == 0) {
            constexpr int i = D0 + J / PER, tm = useE ? J % PER / 3 : 1, q = J % 3;
            dl[J & 1] = sh.left[(x - 1) & 3][i][2 * tm + (q == 2)][lane];
            df[J & 1][0] = sh.frag[(x - 1) & 1][2 * tm + (q == 1)][0][lane];
            df[J & 1][1] = sh.frag[(x - 1) & 1][2 * tm + (q == 1)][1][lane];
          }
          if constexpr (J >= 1 && J <= NSLOT) {
            constexpr int i = D0 + (J - 1) / PER, b = (J - 1) & 1;
            acc[i][rh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, dl[b]), __builtin_bit_cast(bf16x8, df[b][rh]), acc[i][rh], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      u32x4 pe[2][2], pv[2][2];                            // -E and V as bf16 hi, lo: 16 columns as two chunks of eight
      sb_steps<TERMS, 0>(w, d, u, p, dreg, g, -g.zr, a.maxq - g.zr, 0.f, 0.f, pe, between);
      // ---- the update of the next sub-block's piece, the one thing that sub-block waits for.  Its MFMAs run beside the rest of this
      // one's work, the split of V under the products of -E, and the writes to LDS.
      constexpr bool own = update && NEXT < 4;
      u32x4 left[4];
      if constexpr (own) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (q < 2 ? useE : useP) left[q] = sh.left[x & 3][NEXT][q][lane];
      }
      auto product = [&](int tm, int k, const u32x4 (&f)[2][2]) {        // k-th MFMA of a term
        if constexpr (own) {
          const int q = k >> 1, rh = k & 1;
          acc[NEXT][rh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, left[2 * tm + (q == 2)]),
                                                                  __builtin_bit_cast(bf16x8, f[q == 1][rh]), acc[NEXT][rh], 0, 0, 0);
        }
      };
      auto split_v = [&](int k) {                                         // V of columns 2 k and 2 k + 1
        const u32x2 s = sb_split2(w[2 * k], w[2 * k + 1]);
        pv[0][k >> 2][k & 3] = s[0];
        pv[1][k >> 2][k & 3] = s[1];
      };
      sb_to_operand(pe[0]);
      sb_to_operand(pe[1]);
      *reinterpret_cast<f32x4*>(&sh.d[buf][lane][12]) = f32x4{d[12], d[13], d[14], d[15]};
      *reinterpret_cast<u32x2*>(&sh.grid[buf][lane][0]) = u32x2{__float_as_uint(g.sc), __float_as_uint(g.zr)};
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        if (useE) product(0, k, pe);
        __builtin_amdgcn_sched_barrier(0);
        if (k < 4) sh.frag[buf][k >> 1][k & 1][lane] = pe[k >> 1][k & 1];
        split_v(k);
        if (k >= 4) split_v(k + 2);
        __builtin_amdgcn_sched_barrier(0);
      }
      sb_to_operand(pv[0]);
      sb_to_operand(pv[1]);
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        if (useP) product(1, k, pv);
        __builtin_amdgcn_sched_barrier(0);
        if (k < 4) sh.frag[buf][2 + (k >> 1)][k & 1][lane] = pv[k >> 1][k & 1];
        __builtin_amdgcn_sched_barrier(0);
      }
      if (!CLIP && EB < 7 && x + 1 < last_own) load_diag(x + 1);
      sb_barrier();
      if constexpr (own) {
        // the other pieces that cannot wait for the next column steps
#pragma unroll
        for (int i = NEXT + 1; i < sb_first_deferred(EB); ++i) {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (q < 2 ? useE : useP) left[q] = sh.left[x & 3][i][q][lane];
          const u32x4 fr[4][2] = {{pe[0][0], pe[0][1]}, {pe[1][0], pe[1][1]}, {pv[0][0], pv[0][1]}, {pv[1][0], pv[1][1]}};
          sb_piece_update(acc[i], left, fr, useE, useP, [](int) {});
        }
      }
    };
    event(std::integral_constant<int, 0>{});
    event(std::integral_constant<int, 1>{});
    event(std::integral_constant<int, 2>{});
    event(std::integral_constant<int, 3>{});
    event(std::integral_constant<int, 4>{});
    event(std::integral_constant<int, 5>{});
    event(std::integral_constant<int, 6>{});
    event(std::integral_constant<int, 7>{});
    e = last_own;
    __builtin_amdgcn_s_setprio(0);
  }

  // ================= finished
  for (; e < nev; ++e) {
    help_begin(e);
    if (group_starts(e)) search();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    help_end(e);
    sb_barrier();
  }
  help_end(nev);
}

hipError_t launch_near_operands(const float* U, const float* P, int64_t ldh, int n, int first, int count, const SbNear& o, hipStream_t s) {
  hipLaunchKernelGGL(near_operands_kernel, dim3(kSbCols / 64, kSbCols / kSub, 2 * count), dim3(256), 0, s, U, P, ldh, n, first, o);
  return hipGetLastError();
}

template <bool FAST, int TERMS, bool CLIP>
static hipError_t launch_quant_sb_as(const SbArgs& a, hipStream_t s) {
  constexpr int lds = (int)(sizeof(SbShared) + (CLIP ? sizeof(SbClip) : 0));
  static LdsLimitOnce once;                      // per instantiation
  const hipError_t e = once.ensure(reinterpret_cast<const void*>(&quant_sb_kernel<FAST, TERMS, CLIP>), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((quant_sb_kernel<FAST, TERMS, CLIP>), dim3((a.m + 63) / 64), dim3(64 * kSbWaves), lds, s, a);
  return hipGetLastError();
}

template <int TERMS>
static hipError_t launch_quant_sb_terms(const SbArgs& a, hipStream_t s) {
  if (a.clip_steps > 0) return a.fast_rows ? launch_quant_sb_as<true, TERMS, true>(a, s) : launch_quant_sb_as<false, TERMS, true>(a, s);
  return a.fast_rows ? launch_quant_sb_as<true, TERMS, false>(a, s) : launch_quant_sb_as<false, TERMS, false>(a, s);
}

hipError_t launch_quant_sb(const SbArgs& a, hipStream_t s) {
  switch (a.terms) {
    case 3: return launch_quant_sb_terms<3>(a, s);
    case 2: return launch_quant_sb_terms<2>(a, s);
    case 1: return launch_quant_sb_terms<1>(a, s);
    default: return launch_quant_sb_terms<0>(a, s);
  }
}

}  // namespace gptaq
