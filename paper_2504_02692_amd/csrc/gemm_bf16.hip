// bf16 x bf16 -> fp32 MFMA GEMM for gfx950:  C (+)= sum over terms of (sum of cross products) L R^T.
//
// Every dense contraction of the solve goes through this kernel (Algorithm 1 line 2: H and
// dXXT; line 4: the two products of Theorem 4.2; lines 11-12: the lazy trailing update of
// Eq. 18).  Where fp32 operands need more than bf16's 8 bits, an operand is split into bf16
// hi + lo (about 2^-17 relative) and the cross products hi*hi + hi*lo + lo*hi are summed in fp32.
//
// Tiling: a 256-thread workgroup owns a BT x BT tile of C (BT = 256 or 128); its four
// wavefronts sit 2 x 2 and each accumulates a (BT/2)^2 sub-tile with
// v_mfma_f32_32x32x16_bf16 (accumulators in AGPRs).  Operand k-tiles (BT rows x 32 bf16) go
// from global memory straight into LDS (global_load_lds_dwordx4, no VGPR staging) through a
// ring of LDS stages, ahead of the multiply; fragment reads are ds_read_b128 on an
// XOR-swizzled layout and run one k-step ahead of the MFMAs.
//
// Feeding the operands is what bounds this kernel: a CU takes at most ~22 bytes per clock from its L2
// into LDS (measured; less when lines come from HBM), which is about what one 256 x 256 product per
// two operand tiles needs at full MFMA rate.  So operand tiles are shared between cross products: per
// k-tile a term loads its NL left and NR right operand tiles once and multiplies all listed
// (left, right) pairs from them - dXXT's hi and lo halves share the X tile, and the three products of
// a split term need four tiles instead of six.  The loads of a k-tile are issued one by one between
// the MFMAs of an earlier k-tile, and the barriers carry no memory fence, so that loads stay in
// flight across them (see wg_barrier).
#include "common.h"
#include <utility>

namespace gptaq {

template <int KIND> struct KindTraits;
template <> struct KindTraits<0> { static constexpr int NL = 1, NR = 1, NPAIR = 1, NSTAGE = 4; };
template <> struct KindTraits<1> { static constexpr int NL = 2, NR = 1, NPAIR = 2, NSTAGE = 3; };
template <> struct KindTraits<2> { static constexpr int NL = 2, NR = 2, NPAIR = 3, NSTAGE = 2; };
// pair p of a kind: (left index, right index)  (kind 3 has a loop of its own: remainder_loop)
__device__ __forceinline__ constexpr int pair_l(int kind, int p) { return kind == 0 ? 0 : kind == 1 ? p : (p == 2 ? 1 : 0); }
__device__ __forceinline__ constexpr int pair_r(int kind, int p) { return kind == 2 ? (p == 1 ? 1 : 0) : 0; }

// Workgroup barrier without the memory fence of __syncthreads(): that fence makes the compiler drain
// every outstanding global -> LDS load (vmcnt(0)) at each barrier, which would cut the load pipeline
// down to one k-tile.  The waits a barrier needs here are written out by hand before it.
__device__ __forceinline__ void wg_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int N> __device__ __forceinline__ void wait_vm_and_lds() {
  // vmcnt <= N (vmcnt is split over bits 3:0 and 15:14), lgkmcnt == 0, expcnt untouched
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
}

constexpr int kFlagBytes = kMaxRemainderK / kGemmBK;      // kind 3: a byte per k-tile
constexpr int kLds256 = 3 * (3 * 256 * 64 + 256 * 4) + kFlagBytes;    // kind 3: 3 stages x (3 operand tiles, positions), flags (2 x 4 and 4 x 2 tiles are smaller)
constexpr int kLds128 = 3 * (3 * 128 * 64 + 128 * 4) + kFlagBytes;

template <int BT, int KIND, bool MULTI>
__device__ __forceinline__ void tile_loop(const GemmProblem& P, unsigned char* smem, int m0, int n0, int klo, int nk,
                                          f32x16 (&acc)[BT / 64][BT / 64]) {
  using T = KindTraits<KIND>;
  constexpr int NL = T::NL, NR = T::NR, NOP = NL + NR, NSTAGE = T::NSTAGE;
  constexpr int WT = BT / 2, FR = WT / 32;
  constexpr int OPB = BT * 64;           // bytes of one operand k-tile (BT rows x 32 bf16)
  constexpr int STAGE_BYTES = NOP * OPB;
  constexpr int LPW = BT / 64;           // 1 KB wave-loads per operand per wave per k-tile
  constexpr int TL = NOP * LPW;          // loads per k-tile per wave
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int total_it = nk * P.nterm;

  // ---- LDS tile format.  An operand k-tile is BT rows x 32 bf16 (64 B per row).  The LDS of gfx950
  // has 64 banks (256 B per clock), and a ds_read_b128 serves 16 lanes per clock, so 16 consecutive
  // fragment rows of one 16-byte chunk column must land in 16 different 16-byte slots of a 256-byte
  // line.  Four rows share a line; slot = (row & 3) * 4 + (chunk ^ (line & 3)): the four lines that
  // 16 consecutive rows touch use four different XOR values, i.e. disjoint slot sets.
  // Loads go global -> LDS directly: lane l of a wave writes the 16 bytes at LDS base + 16 l, so a
  // wave fills 4 consecutive lines (16 rows) and each lane fetches the (row, chunk) of its slot.
  const int ld_line = lane >> 4;
  const int ld_row = ld_line * 4 + ((lane & 15) >> 2);
  const int ld_chunk = (lane & 3) ^ ld_line;
  // The TL wave loads of a k-tile are issued one at a time, spread between the MFMAs of the k-tile
  // before it (a wave stalls ~50 clocks per 1 KB load it hands to the memory pipeline; in a burst that
  // is time the matrix unit idles).  Past the last k-tile the last one is fetched again into the stage
  // that has just been retired, which keeps the loop and its wait counts free of special cases.
  // The tiles are loaded in order, so the source is a cursor: per-lane pointers to the next tile, moved on
  // by one k-tile after each (recomputed only where the second term starts).
  struct TileSrc {
    const uint16_t* l[NL];
    const uint16_t* r[NR];
    int64_t lstep, rstep;     // 16 rows, in elements
    int64_t lkt, rkt;         // one k-tile, in elements
    unsigned char* st;        // this wave's part of the stage the tile goes to
    int seq;                  // number of the tile in load order (not clamped)
  };
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  auto seek_term = [&](TileSrc& c, int t) {
    const GemmTerm& tm = P.term[t];
    const int64_t kt = klo / kGemmBK;
    const int64_t lo = (int64_t)(m0 + wave * LPW * 16 + ld_row) * tm.ldl + kt * tm.ktl + ld_chunk * 8;
    const int64_t ro = (int64_t)(n0 + wave * LPW * 16 + ld_row) * tm.ldr + kt * tm.ktr + ld_chunk * 8;
#pragma unroll
    for (int o = 0; o < NL; ++o) c.l[o] = tm.L[o] + lo;
#pragma unroll
    for (int o = 0; o < NR; ++o) c.r[o] = tm.R[o] + ro;
    c.lstep = 16 * tm.ldl;
    c.rstep = 16 * tm.ldr;
    c.lkt = tm.ktl;
    c.rkt = tm.ktr;
  };
  // moves the cursor on by one k-tile; `stage` (static) is the stage the new tile goes to
  auto next_tile = [&](TileSrc& c, int stage) {
    ++c.seq;
    c.st = smem + stage * STAGE_BYTES + wave_s * LPW * 1024;
    if (MULTI && c.seq == nk && c.seq < total_it) {
      seek_term(c, 1);
    } else {
      const int64_t ls = c.seq < total_it ? c.lkt : 0, rs = c.seq < total_it ? c.rkt : 0;
#pragma unroll
      for (int o = 0; o < NL; ++o) c.l[o] += ls;
#pragma unroll
      for (int o = 0; o < NR; ++o) c.r[o] += rs;
    }
  };
  // q-th load of the tile: q = j * NOP + o (16-row slab j of operand o)
  auto load_one = [&](const TileSrc& c, int q) {
    const int j = q / NOP, o = q % NOP;
    const uint16_t* src = o < NL ? c.l[o < NL ? o : 0] + j * c.lstep : c.r[o < NL ? 0 : o - NL] + j * c.rstep;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)(c.st + j * 1024 + o * OPB), 16, 0, 0);
  };

  // fragment reads: lane -> row (lane & 31) of a 32-row block, chunk 2 kk + (lane >> 5)
  const int rl = lane & 31, half = lane >> 5;
  const int fr_line = rl >> 2, fr_x = fr_line & 3, fr_hi = (rl & 3) << 2;
  bf16x8 af[2][NL][FR], bfr[2][NR][FR];
  constexpr int NFRAG = NOP * FR;      // fragments per k-step: NL * FR left, then NR * FR right
  struct FragSrc { const unsigned char* lb; const unsigned char* rb; };
  auto frag_src = [&](int stage, int kk) {
    const int off = (fr_hi | ((kk * 2 + half) ^ fr_x)) << 4;
    FragSrc f;
    f.lb = smem + stage * STAGE_BYTES + (wm * (WT / 4) + fr_line) * 256 + off;
    f.rb = smem + stage * STAGE_BYTES + NL * OPB + (wn * (WT / 4) + fr_line) * 256 + off;
    return f;
  };
  auto read_one = [&](const FragSrc& f, int set, int r) {
    if (r < NL * FR) {
      const int o = r / FR, i = r % FR;
      af[set][o][i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(f.lb + o * OPB + i * 8 * 256));
    } else {
      const int o = (r - NL * FR) / FR, i = (r - NL * FR) % FR;
      bfr[set][o][i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(f.rb + o * OPB + i * 8 * 256));
    }
  };
  // The MFMAs of one k-step on fragment set `set`.  Between them, one at a time (so that each is issued
  // in the shadow of a running MFMA instead of holding up the next one): the fragment reads of the other
  // set for the following k-step, and loads q0 .. q1-1 of tile `c`.
  constexpr int NM = T::NPAIR * FR * FR;
  static_assert(TL <= NM && NFRAG <= NM, "at most one load and one fragment read per MFMA");
  auto mfma_step = [&](int set, const FragSrc& f, const TileSrc& c, int q0, int q1) {
#pragma unroll
    for (int p = 0; p < T::NPAIR; ++p)
#pragma unroll
      for (int i = 0; i < FR; ++i)
#pragma unroll
        for (int j = 0; j < FR; ++j) {
          const int m = (p * FR + i) * FR + j, nq = q1 - q0;
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[set][pair_l(KIND, p)][i], bfr[set][pair_r(KIND, p)][j],
                                                              acc[i][j], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          if (m < NFRAG) read_one(f, set ^ 1, m);
          if ((m + 1) * nq / NM > m * nq / NM) load_one(c, q0 + m * nq / NM);
          __builtin_amdgcn_sched_barrier(0);
        }
  };
  // Pipeline: k-tile `it` is multiplied from stage it % NSTAGE.  One barrier per k-tile, in the middle of
  // its MFMAs: it publishes tile it+1 (every wave has waited for its own loads of it: they return in
  // order, so "at most so many outstanding" says which have landed) and retires stage it % NSTAGE, whose
  // last fragments were read before it.  Tile it + NSTAGE goes into that stage: its first HF loads are
  // issued behind the barrier, the rest before the next one, so each has at least a whole k-tile of
  // MFMA time to arrive (half of one with two stages).
  constexpr int HF = NSTAGE >= 3 ? TL / 2 : TL;
  constexpr int PENDING = (NSTAGE - 2) * TL;               // loads of later tiles issued by the barrier
  if (total_it <= 0) return;
  TileSrc c;
  seek_term(c, 0);
  c.seq = 0;
  c.st = smem + wave_s * LPW * 1024;
#pragma unroll
  for (int t = 0; t < NSTAGE - 1; ++t) {
#pragma unroll
    for (int q = 0; q < TL; ++q) load_one(c, q);
    next_tile(c, t + 1);
  }
#pragma unroll
  for (int q = 0; q < HF; ++q) load_one(c, q);
  wait_vm_and_lds<PENDING + HF>();
  wg_barrier();
  {
    const FragSrc f0 = frag_src(0, 0);
#pragma unroll
    for (int r = 0; r < NFRAG; ++r) read_one(f0, 0, r);
  }
  // NSTAGE k-tiles per trip, so that every stage number below is a constant (LDS addresses and DMA targets
  // become immediates and scalars instead of per-iteration vector arithmetic)
  for (int it0 = 0; it0 < total_it; it0 += NSTAGE) {
#pragma unroll
    for (int sg = 0; sg < NSTAGE; ++sg) {
      if (it0 + sg < total_it) {
        __builtin_amdgcn_sched_barrier(0);
        mfma_step(0, frag_src(sg, 1), c, HF, TL);
        __builtin_amdgcn_sched_barrier(0);
        wait_vm_and_lds<PENDING>();
        wg_barrier();
        __builtin_amdgcn_sched_barrier(0);
        next_tile(c, sg);                                   // tile it + NSTAGE goes where tile it was
        // (behind the last k-tile these fragment reads fetch a stale stage and nobody uses them)
        mfma_step(1, frag_src((sg + 1) % NSTAGE, 0), c, 0, HF);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  wait_vm_and_lds<0>();   // the surplus loads past the last k-tile
}

// The products of remainder_loop are assembly: v_smfmac's result is its accumulator, and from the builtins the compiler made copies of
// accumulators, for which there are no registers (1.8 KB of scratch a lane).  It does not look into assembly: an operand must not have
// been written by a vector instruction less than two wait states before (a nop stands for them where positions are moved; hi comes
// from LDS), and what reads the accumulators as registers waits for the last product (settle); that one product adds to what another
// has just written is the hardware's to order.  tests/test_mfma_hazards.py looks at every build.
__device__ __forceinline__ void dense_product(f32x16& acc, bf16x8 l, bf16x8 x) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(l), "v"(x));
}
constexpr uint16_t kPositions01 = 0x4444, kPositions23 = 0xEEEE;          // the first two of every four tokens, and the last two
__device__ __forceinline__ void sparse_product(f32x16& acc, bf16x8 lo, bf16x16 x, uint16_t pos) {      // 32 tokens
  asm volatile("s_nop 1\n\tv_smfmac_f32_32x32x32_bf16 %0, %1, %2, %3" : "+a"(acc) : "v"(lo), "v"(x), "v"(pos));
}
// lo2's products of a row of blocks, if on != 0 (the branch is inside, so that no accumulator has two ways to come from)
__device__ __forceinline__ void sparse_products_if(int on, f32x16 (&a)[2], bf16x8 lo, const bf16x16 (&x)[2]) {
  asm volatile("s_cmp_eq_u32 %6, 0\n\ts_cbranch_scc1 .Lnone%=\n\ts_nop 1\n\t"
               "v_smfmac_f32_32x32x32_bf16 %0, %2, %3, %5\n\tv_smfmac_f32_32x32x32_bf16 %1, %2, %4, %5\n.Lnone%=:"
               : "+a"(a[0]), "+a"(a[1]) : "v"(lo), "v"(x[0]), "v"(x[1]), "v"(kPositions23), "s"(on) : "scc");
}
__device__ __forceinline__ void sparse_products_if(int on, f32x16 (&a)[4], bf16x8 lo, const bf16x16 (&x)[4]) {
  asm volatile("s_cmp_eq_u32 %10, 0\n\ts_cbranch_scc1 .Lnone%=\n\ts_nop 1\n\t"
               "v_smfmac_f32_32x32x32_bf16 %0, %4, %5, %9\n\tv_smfmac_f32_32x32x32_bf16 %1, %4, %6, %9\n\t"
               "v_smfmac_f32_32x32x32_bf16 %2, %4, %7, %9\n\tv_smfmac_f32_32x32x32_bf16 %3, %4, %8, %9\n.Lnone%=:"
               : "+a"(a[0]), "+a"(a[1]), "+a"(a[2]), "+a"(a[3])
               : "v"(lo), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(kPositions23), "s"(on) : "scc");
}
__device__ __forceinline__ void settle(f32x16& acc) { asm volatile("s_nop 15\n\ts_nop 7" : "+a"(acc)); }

// f of the numbers 0 .. N - 1, as types
template <class F, int... I> __device__ __forceinline__ void static_for_each(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void static_for(F&& f) { static_for_each(f, std::make_integer_sequence<int, N>{}); }

// 16 or 4 bytes a lane, one lane's behind the other's from dst on; OFFSET counts on both sides
template <int OFFSET> __device__ __forceinline__ void load_to_lds16(const unsigned char* src, unsigned char* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)dst, 16, OFFSET, 0);
}
__device__ __forceinline__ void load_to_lds4(const unsigned char* src, unsigned char* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)dst, 4, 0, 0);
}

__device__ __align__(16) unsigned char zeros[4096];         // stands in for lo2 of a block that has none

// Which of remainder_loop's two forms by blocks: from so many dense 32 x 32 blocks per k-tile on (of 8 and of 4, the mean over the k-tiles of a
// tile) lo2's products are taken with the rest.  Us with branches / without, of 32768 tokens, upper form: 4096 columns, 69 % dense: 1550 / 1606, 96 %: 1629 /
// 1605; 11008 columns 9695 / 9980, 10030 / 9960.  A workgroup alone on its CU waits for the branches, which another one does not hide: with
// 128-tiles 2048 columns, 14 %: 596 / 600, 38 %: 644 / 598 (and, with two to a CU, 2736 columns in the full form 1249 / 1295).
constexpr int kMany256 = 7, kMany128 = 1;

// Kind 3: acc += (hi + lo) X^T, hi and X bf16 operands as above, lo the remainder of hi, of which few entries are not zero (GemmTerm says
// how it is stored).  lo1 takes a v_smfmac_f32_32x32x32_bf16 per 32 x 32 block and k-tile, at twice the rate of a dense product; lo2 of
// a dense block a second one.  Bound by its operand bytes (41 KB per 32 tokens of a 256-tile for 1536 clocks of products, 49 for 2048 where
// all blocks are dense) and by the power-limited clock, so little is done beside the products: a block's positions are ready to use, and
// its lo2 is fetched, and with 256-tiles multiplied, behind a branch of that block alone.  (With the positions of a dense block's values among the words of
// lo2, a word of two for each four tokens, taking them out was 100 vector instructions a k-tile: 4096 columns and 32768 tokens 1974 us where all blocks are
// dense, so 1640; dense operands 1620.)
template <int BT>
__device__ __forceinline__ void remainder_loop(const GemmProblem& P, unsigned char* smem, int m0, int n0, int nk, f32x16 (&acc)[BT / 64][BT / 64]) {
  constexpr int NSTAGE = 3, WT = BT / 2, FR = WT / 32;
  constexpr int OPB = BT * 64, LOB = BT * 32, GROUP = 4096;            // bytes of a k-tile of hi or X, of lo1 or lo2; of 128 rows of R[1]
  constexpr int LO1 = 2 * OPB, LO2 = LO1 + LOB, POS = LO2 + LOB, STAGE_BYTES = POS + BT * 4, FLAGS = NSTAGE * STAGE_BYTES;
  constexpr int LPW = BT / 64, LPWL = LOB / 4096;           // 1 KB loads per wave and k-tile: of hi or X, of lo1 or lo2
  if (nk <= 0) return;                                      // (nk is even)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const GemmTerm& tm = P.term[0];
  typedef const unsigned char* Bytes;
  const bool rows = P.lo_rows != 0;
  const int64_t kt = tm.ktl * 2;                            // bytes per k-tile of hi or X

  // A source is a base that the wavefront shares and a lane's offset.  hi, X and lo by rows: the tile format of tile_loop.  lo1 and lo2: a block has 64
  // slots of 16 bytes in LDS, those of row r at 2 r and 2 r + 1, exchanged in every other eight rows, so that 16 lanes that read one half of
  // 16 rows meet 16 different slots of a 256-byte line.
  const uint32_t at64 = ((lane >> 4) * 4 + ((lane & 15) >> 2)) * 64 + ((lane & 3) ^ (lane >> 4)) * 16;
  const int piece = lane ^ (lane >> 4 & 1);                 // of a block's 64 times 16 bytes
  const uint32_t at32 = piece * 16;
  const uint32_t lo2_step = piece == 0 ? 16 : piece < 9 ? 128 : 880;      // from block to block of R[1]
  const uint32_t at_lo2 = (piece == 0 ? 0 : piece < 9 ? 48 + 16 * piece : 432 + 16 * piece) + (wave & (4 / LPWL - 1)) * LPWL * lo2_step;
  // the positions that a wavefront fetches, 256 bytes of a group's 512 (with 128 rows two fetch the same)
  const int pos_part = BT == 256 ? wave_s : wave_s & 1;
  struct TileSrc {
    Bytes hi, x, lo, lo2;
    int st, seq;                                            // where in LDS the tile goes, and its number in load order (not clamped)
  } c;
  c.hi = (Bytes)tm.L[0] + (int64_t)m0 * 64 + wave_s * (LPW * 1024);
  c.x = (Bytes)tm.R[0] + (int64_t)n0 * 64 + wave_s * (LPW * 1024);
  c.lo = (Bytes)tm.L[1] + (rows ? (int64_t)m0 * 64 + wave_s * (LPW * 1024) : (int64_t)m0 * 32 + wave_s * (LPWL * 1024));
  c.lo2 = (Bytes)tm.R[1] + (int64_t)m0 * 32;
  c.st = 0;
  c.seq = 0;
  auto next_tile = [&](int stage_at) {
    ++c.seq;
    c.st = stage_at;
    const int64_t step = c.seq < nk ? kt : 0;
    c.hi += step;
    c.x += step;
    c.lo += rows ? step : step / 2;
    c.lo2 += step / 2;
  };
  // 1 KB, number `slab` of those that a wavefront fetches of an operand
  auto to_lds = [&](Bytes base, uint32_t at, int lds, auto slab) { load_to_lds16<decltype(slab)::value * 1024>(base + (uint64_t)at, smem + lds); };
  auto load_hi_x = [&](auto number) {                       // (in turn)
    constexpr int q = decltype(number)::value;
    if constexpr (q & 1) to_lds(c.x, at64, c.st + OPB + wave_s * (LPW * 1024), std::integral_constant<int, q / 2>{});
    else to_lds(c.hi, at64, c.st + wave_s * (LPW * 1024), std::integral_constant<int, q / 2>{});
  };
  auto load_lo_rows = [&](auto slab) { to_lds(c.lo, at64, c.st + LO1 + wave_s * (LPW * 1024), slab); };
  auto load_lo1 = [&](auto slab) { to_lds(c.lo, at32, c.st + LO1 + wave_s * (LPWL * 1024), slab); };
  auto load_lo2 = [&](Bytes base, auto number) {            // of block `number` of the wavefront's LPWL
    constexpr int p = decltype(number)::value;
    to_lds(base, at_lo2 + p * lo2_step, c.st + LO2 + (wave_s * LPWL + p) * 1024, std::integral_constant<int, 0>{});
  };
  auto lo2_of_wave = [&]() { return c.lo2 + (wave_s * LPWL >> 2) * GROUP; };
  auto load_positions = [&]() {
    load_to_lds4(c.lo2 + (pos_part >> 1) * GROUP + 64 + (pos_part & 1) * 256 + (uint64_t)(uint32_t)(lane * 4), smem + c.st + POS + pos_part * 256);
  };

  const int rl = lane & 31, half = lane >> 5;
  const int fr_line = rl >> 2, fr_x = fr_line & 3, fr_hi = (rl & 3) << 2;
  auto frag = [&](const unsigned char* st, int kk, int i) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(st + i * 2048 + fr_line * 256 + ((fr_hi | ((kk * 2 + half) ^ fr_x)) << 4)));
  };
  const int lo_at = wm * (FR * 1024) + (2 * rl + (half ^ (rl >> 3 & 1))) * 16, pos_at = POS + wm * (FR * 128) + rl * 4 + half * 2;
  auto lo_frag = [&](const unsigned char* st, int i) { return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(st + lo_at + i * 1024)); };
  unsigned char* flags = smem + FLAGS;
  auto blocks_of = [&](int f) { return (f >> (wave_s >> 1) * FR) & ((1 << FR) - 1); };      // this wavefront's
  int fl0 = 0, fl1 = 0, fl2 = 0, mark = 0;                                  // the dense blocks of the k-tiles it, it + 1, it + 2, and of the one behind them

  // Pipeline: one barrier per k-tile `it`, behind which tile it + 1 is in LDS and tile it in registers.  A 32-row block's products
  // (hi in two k-steps, lo1, lo2) are taken one after the other.  Between them, one at a time, the fragments of tile it + 1 are read: with
  // 256-tiles those of a block into its registers of tile it while the next block is multiplied (the last block's into two sets
  // in turn), with 128-tiles there are two sets for all; and tile it + NSTAGE is requested.
  // ALWAYS: lo2 is fetched (where a block has none, from zeros) and multiplied with the rest; else behind a branch per block.
  // ROWS: lo by rows.  Whether a row is one of a sparse block, and its positions then, come out of the first words of its lo2; lo2 is multiplied
  // where one of the 32 rows is not.
  auto run = [&](auto layout, auto form) {
    constexpr bool ROWS = decltype(layout)::value, ALWAYS = decltype(form)::value;
    constexpr int G = (ALWAYS ? 4 : 3) * FR, NSLOT = G * FR, LOADS = 2 * LPW + (ROWS ? LPW : LPWL + 1 + (ALWAYS ? LPWL : 0)), LOAD_SLOTS = NSLOT - 4;
    constexpr bool TWO = FR == 2;                           // two whole sets
    // lo2 of a k-tile's two blocks behind them, with one branch for both where it is rare (2736 columns full 1145 us, so 1108)
    constexpr bool LAST = TWO && !ROWS && !ALWAYS;
    constexpr int SETS = TWO ? 2 * FR : FR + 1;
    constexpr int PER = ROWS ? 6 : 7, ROUNDS = TWO ? 1 : FR, ROUND_SLOTS = NSLOT / ROUNDS;         // reads of a block (with those of X that come along)
    constexpr int READS = PER * FR / ROUNDS, READ_SLOTS = TWO ? NSLOT - 1 : ROUND_SLOTS - 2;
    bf16x8 a[SETS][2], b[2][2][FR], l1[SETS], l2[SETS];
    uint16_t pos[SETS], p = 0;                              // (16 bits: the compiler would clear the others otherwise)
    int on = 0;                                             // whether the block that is multiplied is dense; p: its positions
    auto set_of = [](int i, int s) { return TWO ? 2 * i + s : i < FR - 1 ? i : FR - 1 + s; };
    // of block i of the k-tile at st, to set t
    auto read_item = [&](const unsigned char* st, int i, int t, int item) {
      if (item == 0) l1[t] = ROWS ? frag(st + LO1 + wm * (WT * 64), 0, i) : lo_frag(st + LO1, i);
      else if (item == 1) l2[t] = ROWS ? frag(st + LO1 + wm * (WT * 64), 1, i) : lo_frag(st + LO2, i);
      else if (item < 4) a[t][item - 2] = frag(st + wm * (WT * 64), item - 2, i);
      else pos[t] = *reinterpret_cast<const uint16_t*>(st + pos_at + i * 128);
    };
    auto read_x = [&](const unsigned char* st, int s, int k) { b[s][k / FR][k % FR] = frag(st + OPB + wn * (WT * 64), k / FR, k % FR); };
#pragma unroll
    for (int i = 0; i < FR; ++i) {
#pragma unroll
      for (int item = 0; item < PER - 2; ++item) read_item(smem, i, set_of(i, 0), item);
#pragma unroll
      for (int k = 0; k < 2; ++k) read_x(smem, 0, 2 * i + k);
    }
    int cur = 0;                                            // where the stage of this k-tile begins
    for (int it0 = 0; it0 < nk; it0 += 2) {
      static_for<2>([&](auto parity) {
        constexpr int s = decltype(parity)::value;
        const int it = it0 + s, nxt = cur == (NSTAGE - 1) * STAGE_BYTES ? 0 : cur + STAGE_BYTES;
        const unsigned char* nx = smem + nxt;
        auto both = [&](int j) { return __builtin_shufflevector(b[s][0][j], b[s][1][j], 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15); };
        __builtin_amdgcn_sched_barrier(0);
        wait_vm_and_lds<LOADS>();                           // (all but what the k-tile before has requested: so many at least)
        wg_barrier();
        __builtin_amdgcn_sched_barrier(0);
        const int now = blocks_of(fl0);
        static_for<NSLOT>([&](auto slot) {
          constexpr int m = decltype(slot)::value, i = m / G, q = m % G, ph = q / FR, j = m % FR;
          const int t = set_of(i, s);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (ph < 2) dense_product(acc[i][j], a[t][ph], b[s][ph][j]);
          else if constexpr (ph == 2) sparse_product(acc[i][j], l1[t], both(j), p);
          else sparse_product(acc[i][j], l2[t], both(j), kPositions23);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (q == FR) {
            if constexpr (ROWS) {
              u32x4 w = __builtin_bit_cast(u32x4, l2[t]);
              const uint32_t x = w[0] ^ kRowMark;
              const bool mark = x < 0x10000u;
              p = mark ? (uint16_t)x : kPositions01;
              w[0] = mark ? 0u : w[0];
              l2[t] = __builtin_bit_cast(bf16x8, w);
              const uint64_t those = __ballot(!mark);
              on = __builtin_amdgcn_readfirstlane((uint32_t)those | (uint32_t)(those >> 32));
            } else {
              on = now >> i & 1;
              p = on ? kPositions01 : pos[t];
            }
          }
          // (behind the last k-tile: a stale stage, not used)
          constexpr int round = m / ROUND_SLOTS, rq = m % ROUND_SLOTS;
          constexpr int r0 = (rq * READS + READ_SLOTS - 1) / READ_SLOTS, r1 = ((rq + 1) * READS + READ_SLOTS - 1) / READ_SLOTS;
          static_for<(r0 < READS ? (r1 < READS ? r1 : READS) - r0 : 0)>([&](auto number) {
            constexpr int n = r0 + decltype(number)::value, item = n % PER, x = item - (PER - 2);
            constexpr int block = TWO ? n / PER : (round + FR - 1) % FR;
            if constexpr (x < 0) read_item(nx, block, set_of(block, s ^ 1), item);
            else read_x(nx, s ^ 1, 2 * (TWO ? block : round) + x);
          });
          if constexpr (!ROWS && m == 1) {
            const int f = __builtin_amdgcn_readfirstlane(mark);
            fl0 = fl1;
            fl1 = fl2;
            fl2 = c.seq < nk ? f : 0;
            if constexpr (!ALWAYS) static_for<LPWL>([&](auto slab) { if (fl2 >> (wave_s * LPWL + decltype(slab)::value) & 1) load_lo2(lo2_of_wave(), slab); });
          }
          if constexpr (!ROWS && m == NSLOT / 2) mark = flags[min(it + NSTAGE + 1, nk - 1)];
          constexpr int l = m - 2, q0 = l * LOADS / LOAD_SLOTS;
          if constexpr (l >= 0 && l < LOAD_SLOTS && q0 < (l + 1) * LOADS / LOAD_SLOTS) {
            constexpr int w = q0 - 2 * LPW, w2 = w - LPWL;
            if constexpr (w < 0) load_hi_x(std::integral_constant<int, q0>{});
            else if constexpr (ROWS) load_lo_rows(std::integral_constant<int, w>{});
            else if constexpr (q0 == LOADS - 1) load_positions();
            else if constexpr (w2 < 0) load_lo1(std::integral_constant<int, w>{});
            else load_lo2(fl2 >> (wave_s * LPWL + w2) & 1 ? lo2_of_wave() : (Bytes)zeros, std::integral_constant<int, w2>{});
          }
          if constexpr (!ALWAYS && !LAST && q == G - 1) {
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (FR == 4) sparse_products_if(on, acc[i], l2[t], {both(0), both(1), both(2), both(3)});
            else sparse_products_if(on, acc[i], l2[t], {both(0), both(1)});
            __builtin_amdgcn_sched_barrier(0);
          }
          if constexpr (m == NSLOT - 1) { next_tile(nxt); cur = nxt; }
        });
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (LAST) {
          if (__builtin_expect(now != 0, 0)) {
#pragma unroll
            for (int i = 0; i < FR; ++i) sparse_products_if(now >> i & 1, acc[i], l2[set_of(i, s)], {both(0), both(1)});
          }
        }
      });
    }
    wait_vm_and_lds<0>();   // the surplus loads past the last k-tile
#pragma unroll
    for (int i = 0; i < FR; ++i)
#pragma unroll
      for (int j = 0; j < FR; ++j) settle(acc[i][j]);
  };

  static_for<NSTAGE>([&](auto t) {                          // (lo2 too: which blocks are dense is not known yet)
    static_for<2 * LPW>(load_hi_x);
    if (rows) {
      static_for<LPW>(load_lo_rows);
    } else {
      static_for<LPWL>(load_lo1);
      static_for<LPWL>([&](auto number) { load_lo2(lo2_of_wave(), number); });
      load_positions();
    }
    next_tile((decltype(t)::value + 1) % NSTAGE * STAGE_BYTES);
  });
  if (rows) {
    wait_vm_and_lds<0>();
    wg_barrier();
    run(std::true_type{}, std::false_type{});
    return;
  }
  // which blocks of each k-tile are dense, from their heads: a bit per block
  for (int k = tid; k < nk; k += 256) {
    const uint32_t* head = reinterpret_cast<const uint32_t*>((Bytes)tm.R[1] + (int64_t)k * (kt / 2) + (int64_t)m0 * 32);
    int f = 0;
#pragma unroll
    for (int b = 0; b < BT / 32; ++b) f |= head[(b >> 2) * (GROUP / 4) + (b & 3) * 4] != kSparseMark ? 1 << b : 0;
    flags[k] = (unsigned char)f;
  }
  wait_vm_and_lds<0>();
  wg_barrier();
  int marked = 0;                                           // dense blocks
  for (int k = 0; k < nk; k += 64) {
    const int f = k + lane < nk ? flags[k + lane] : 0;
#pragma unroll
    for (int b = 0; b < BT / 32; ++b) marked += __builtin_popcountll(__ballot(f >> b & 1));
  }
  fl0 = __builtin_amdgcn_readfirstlane(flags[0]);
  fl1 = __builtin_amdgcn_readfirstlane(flags[1]);
  fl2 = __builtin_amdgcn_readfirstlane(flags[min(2, nk - 1)]);
  mark = flags[min(NSTAGE, nk - 1)];
  if (marked > nk * (BT == 256 ? kMany256 : kMany128)) {
    // (the first k-tiles have been fetched as they are)
#pragma unroll
    for (int t = 0; t < NSTAGE; ++t)
#pragma unroll
      for (int p = 0; p < LPWL; ++p)
        if (!((t == 0 ? fl0 : t == 1 ? fl1 : fl2) >> (wave_s * LPWL + p) & 1))
          *reinterpret_cast<u32x4*>(smem + t * STAGE_BYTES + LO2 + (wave_s * LPWL + p) * 1024 + lane * 16) = u32x4{0, 0, 0, 0};
    wait_vm_and_lds<0>();
    wg_barrier();
    run(std::false_type{}, std::true_type{});
  } else {
    run(std::false_type{}, std::false_type{});
  }
}

// A wave-uniform value that is to stay in scalar registers (the compiler would otherwise choose between the two problems of a
// batch again at every use).
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t uniform(int64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x), hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// C as a buffer: an element is addressed by a lane offset, a scalar offset and an immediate, all in bytes
struct TileBuffer {
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ __forceinline__ TileBuffer(float* base) : rsrc(__builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00020000)) {}
  __device__ __forceinline__ float load(uint32_t lane, uint32_t scalar) const {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, lane, scalar, 0));
  }
  __device__ __forceinline__ void store(float x, uint32_t lane, uint32_t scalar) const {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), rsrc, lane, scalar, 0);
  }
};

// The accumulators of a BT x BT tile at (m0, n0) to C.
// An element is addressed as (lane offset) + (scalar offset of its row) + (immediate), one instruction each; at the edge of the
// matrix, where a row or a column lies outside, its load reads the tile's first element instead and its store is masked.  With a
// branch per element and 64-bit products per address, ~35 instructions each, a 256-tile took ~45 us here: accumulate_upper at
// n = 4096, where 16 of the 256 CUs have two tiles, took 115 us for 64 tokens and 197 us for 2048; so 56 and 136 (with the sparse remainder and
// H's last tiles as quarters 32 and 105).
// For C += acc the loads run two pieces (of eight rows per half wave) ahead of the stores.  Rows so far apart that a tile is
// out of reach of 32-bit offsets take 64-bit addresses (WIDE).
template <int BT, int MODE, bool EDGE, bool WIDE>
__device__ __forceinline__ void store_tile_as(float* C, int64_t ldc, int M, int N, int run_mode, int m0, int n0,
                                              const f32x16 (&acc)[BT / 64][BT / 64]) {
  constexpr int WT = BT / 2, FR = WT / 32, NC = 2 * FR, AHEAD = WIDE ? 0 : EDGE ? 1 : 2;
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));        // (what follows is not to be kept in registers through the main loop)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row0 = m0 + (wave >> 1) * WT, col0 = n0 + (wave & 1) * WT;               // the wavefront's first element
  const int lrow = 4 * (lane >> 5), lcol = lane & 31;                                // and the lane's, from there
  const int mrem = M - row0 - lrow, nrem = N - col0 - lcol, above = row0 + lrow - col0 - lcol;
  const int store_mode = MODE >= 0 ? MODE : run_mode;
  if (EDGE && (row0 >= M || col0 >= N)) return;
  float* base = C + (int64_t)row0 * ldc + col0;
  const TileBuffer buf(base);
  const uint32_t ld4 = (uint32_t)ldc * 4u, first = (uint32_t)lrow * ld4 + (uint32_t)lcol * 4u;
  auto row = [](int c, int v) { return (c >> 1) * 32 + 8 * (2 * (c & 1) + (v >> 2)) + (v & 3); };
  float old[AHEAD + 1][8][FR];
  auto request = [&](int c) {
#pragma unroll
    for (int v = 0; v < 8; ++v)
#pragma unroll
      for (int j = 0; j < FR; ++j) {
        const int r = row(c, v);
        const bool in = !EDGE || (r < mrem && 32 * j < nrem);
        float& x = old[c % (AHEAD + 1)][v][j];
        if (WIDE) x = in ? base[(int64_t)(lrow + r) * ldc + lcol + 32 * j] : 0.f;
        else if (EDGE) x = buf.load(in ? first + r * ld4 + 128 * j : 0u, 0u);
        else x = buf.load(first + 128 * j, r * ld4);
      }
    __builtin_amdgcn_sched_barrier(0);
  };
  if (store_mode == 0) {
#pragma unroll
    for (int c = 0; c < AHEAD; ++c) request(c);
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    if (store_mode == 0 && c + AHEAD < NC) request(c + AHEAD);
#pragma unroll
    for (int v = 0; v < 8; ++v) {
      const int r = row(c, v);
      if (EDGE && r >= mrem) continue;
#pragma unroll
      for (int j = 0; j < FR; ++j) {
        if (EDGE && 32 * j >= nrem) continue;
        const float a = acc[c >> 1][j][8 * (c & 1) + v];
        const float x = store_mode == 0 ? old[c % (AHEAD + 1)][v][j] + a : run_mode == 1 || 32 * j - r > above ? a : 0.f;
        if (WIDE) base[(int64_t)(lrow + r) * ldc + lcol + 32 * j] = x;
        else if (EDGE) buf.store(x, first + r * ld4 + 128 * j, 0u);
        else buf.store(x, first + 128 * j, r * ld4);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}
template <int BT>
__device__ __forceinline__ void store_tile(float* C, int64_t ldc, int M, int N, int store_mode, int m0, int n0,
                                           const f32x16 (&acc)[BT / 64][BT / 64]) {
  if (ldc >= (1 << 21)) store_tile_as<BT, -1, true, true>(C, ldc, M, N, store_mode, m0, n0, acc);
  else if (m0 + BT > M || n0 + BT > N) store_tile_as<BT, -1, true, false>(C, ldc, M, N, store_mode, m0, n0, acc);
  else if (store_mode == 0) store_tile_as<BT, 0, false, false>(C, ldc, M, N, store_mode, m0, n0, acc);
  else store_tile_as<BT, 2, false, false>(C, ldc, M, N, store_mode, m0, n0, acc);
}

// What lies above the diagonal of C = acc, 0 elsewhere, split into bf16 hi and lo as the left operand of another product (k-tile-major, a
// multiple of the tile in rows and columns), instead of C: entries past the matrix are zeros already.
// Saves a pass over the result: 5 / 17 / 90 us at n = 512 / 4096 / 11008.  (Addressed as in store_tile.)
template <int BT>
__device__ __forceinline__ void store_operand(const GemmProblem& P, int m0, int n0, const f32x16 (&acc)[BT / 64][BT / 64]) {
  constexpr int WT = BT / 2, FR = WT / 32;
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row0 = m0 + (wave >> 1) * WT, col0 = n0 + (wave & 1) * WT;               // the wavefront's first element
  const int64_t first = uniform((int64_t)(col0 >> 5) * P.ldc * 32 + (int64_t)row0 * 32);
  const TileBuffer hi(reinterpret_cast<float*>(P.out_hi + first)), lo(reinterpret_cast<float*>(P.out_lo + first));
  const int lrow = 4 * (lane >> 5), above = row0 + lrow - col0 - (lane & 31);
  const uint32_t at = (uint32_t)(lrow * 64 + (lane & 31) * 2), kt = (uint32_t)uniform(P.ldc) * 64u;
#pragma unroll
  for (int i = 0; i < FR; ++i)
#pragma unroll
    for (int j = 0; j < FR; ++j) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int r = 32 * i + 8 * (v >> 2) + (v & 3);
        const float x = 32 * j - r > above ? acc[i][j][v] : 0.f;
        const __bf16 h = (__bf16)x;
        const __bf16 l = (__bf16)(x - (float)h);
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, h), hi.rsrc, at, j * kt + 64 * r, 0);
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, l), lo.rsrc, at, j * kt + 64 * r, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
}

// Tile row and column of tile number `id` of a problem.
__device__ __forceinline__ void tile_position(const GemmProblem& P, int id, int& tm, int& tn) {
  // Tiles are numbered in groups of GROUP tile rows, column by column inside a group, so the workgroups
  // an XCD runs side by side form a GROUP x 8 patch that shares GROUP left and 8 right operand tiles.
  constexpr int GROUP = 4;
  if (P.tile_mode == 2) {
    // only the tiles with tn >= tm exist: a group holds a small triangle, then full columns
    const int T = P.tiles_n;
    int first = 0, gs, tri;
    for (;;) {
      gs = min(GROUP, T - first);
      tri = gs * (gs + 1) / 2;
      const int cnt = tri + gs * (T - first - gs);
      if (id < cnt) break;
      id -= cnt;
      first += gs;
    }
    if (id < tri) {
      int c = 0;
      while (id > c) { id -= c + 1; ++c; }
      tm = first + id;
      tn = first + c;
    } else {
      id -= tri;
      tn = first + gs + id / gs;
      tm = first + id % gs;
    }
  } else {
    const int width = GROUP * P.tiles_n;
    const int g = id / width, first = g * GROUP;
    const int gsz = min(P.tiles_m - first, GROUP);
    const int r = id - g * width;
    tm = first + r % gsz;
    tn = r / gsz;
  }
}

// A part's BT x BT tile of sums as the accumulators hold it: 16 bytes of a lane are registers 4 v .. 4 v + 3 of a 32 x 32 block (four
// rows of one column), a wavefront's 1 KB one after the other.
template <int BT>
__device__ __forceinline__ void store_partial(float* dst, const f32x16 (&acc)[BT / 64][BT / 64]) {
  constexpr int FR = BT / 64;
  u32x4* out = reinterpret_cast<u32x4*>(dst) + (threadIdx.x >> 6) * (FR * FR * 256) + (threadIdx.x & 63);
#pragma unroll
  for (int i = 0; i < FR; ++i)
#pragma unroll
    for (int j = 0; j < FR; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        out[((i * FR + j) * 4 + v) * 64] = u32x4{__float_as_uint(acc[i][j][4 * v]), __float_as_uint(acc[i][j][4 * v + 1]),
                                                 __float_as_uint(acc[i][j][4 * v + 2]), __float_as_uint(acc[i][j][4 * v + 3])};
}

// One BT x BT tile of C: tile number `wid` of the batch (see the numbering below).
template <int BT, bool CAPPED, bool SPLIT, bool REMAINDER, bool OPERAND>
__device__ __forceinline__ void gemm_tile(const GemmBatch& b, unsigned char* smem, int wid) {
  constexpr int WT = BT / 2;             // wave tile edge
  constexpr int FR = WT / 32;            // 32x32 MFMA blocks per wave tile edge

  // ---- which tile.  Workgroups are dealt round-robin to the 8 XCDs; inside each problem, give every
  // XCD one contiguous run of tiles so that they share operand tiles in that XCD's L2, and so that
  // every XCD gets the same share of each problem (the problems differ in K).
  int id = wid;
  int pi = 0;
  int ntile = b.ntiles[0];
  if (id >= ntile) { pi = 1; id -= ntile; ntile = b.ntiles[1]; }
  const GemmProblem& P = b.p[pi];
  // Quarters of the last tiles of the second problem, behind its whole ones: a CU that has nothing more to do takes one, and the launch
  // ends sooner.  An element's products are added in the same order as in a whole tile.
  if constexpr (REMAINDER && BT == 256) {
    const int whole = ntile - 4 * P.quartered;
    if (pi == 1) {
      if (id >= whole) {
        int q = id - whole, tm, tn;
        q = (q & 7) * (P.quartered >> 1) + (q >> 3);                                  // (an even number: neighbours on one XCD)
        tile_position(P, whole + (q >> 2), tm, tn);
        const int m0 = uniform(tm * 256 + (q & 2) * 64), n0 = uniform(tn * 256 + (q & 1) * 128);
        if (m0 > n0) return;                                                          // (below the diagonal)
        f32x16 acc[2][2];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[i >> 1][i & 1][v] = 0.f;
        tile_loop<128, 0, false>(P, smem, m0, n0, 0, P.K / kGemmBK, acc);
        store_tile<128>(P.C, uniform(P.ldc), uniform(P.M), uniform(P.N), uniform(P.store_mode), m0, n0, acc);
        return;
      }
      ntile = whole;
    }
  }
  if (!P.deal) {
    const int per = ntile >> 3, rem = ntile & 7, xcd = id & 7, loc = id >> 3;
    id = xcd < rem ? xcd * (per + 1) + loc : rem * (per + 1) + (xcd - rem) * per + loc;
  } else if (id < (ntile & ~31)) {
    // With triangular k ranges a contiguous run per XCD would give one XCD the long tiles and another the short ones.
    // Here every XCD takes four consecutive tiles (the four tile rows of one column of a group) out of each 32, so
    // each gets the same mix of lengths, and the 32 workgroups it runs side by side still share four left tiles.
    const int xcd = id & 7, loc = id >> 3;
    id = (((loc >> 2) << 3) + xcd) * 4 + (loc & 3);
  }
  // Split along K: the tiles of the first part of K, then those of the second, ..., so that what runs side by side shares operands.
  const int nt = SPLIT ? ntile / P.split : ntile, part = SPLIT ? id / nt : 0;
  id -= part * nt;
  int tm, tn;
  tile_position(P, id, tm, tn);
  const int m0 = uniform(tm * BT), n0 = uniform(tn * BT);

  const bool skipped = P.tile_mode == 1 && n0 + BT <= m0;
  int klo = 0, khi = P.K;
  if (P.k_mode == 1) klo = min(n0, P.K);
  if (P.k_mode == 2) { klo = min(m0, P.K); khi = min(P.K, n0 + BT); }
  if (SPLIT && P.split > 1) {            // (k_mode 0)
    const int kt = P.K / kGemmBK;
    klo = (int)((int64_t)kt * part / P.split) * kGemmBK;
    khi = (int)((int64_t)kt * (part + 1) / P.split) * kGemmBK;
  }
  const int nk = (skipped || khi <= klo) ? 0 : (khi - klo) / kGemmBK;

  f32x16 acc[FR][FR];
#pragma unroll
  for (int i = 0; i < FR; ++i)
#pragma unroll
    for (int j = 0; j < FR; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  if constexpr (REMAINDER) {
    if (P.kind == 0) tile_loop<BT, 0, false>(P, smem, m0, n0, klo, nk, acc);
    else remainder_loop<BT>(P, smem, m0, n0, nk, acc);
  } else if constexpr (CAPPED) {       // (kind 2 alone: launch_gemm refuses others)
    if (P.nterm > 1) tile_loop<BT, 2, true>(P, smem, m0, n0, klo, nk, acc);
    else tile_loop<BT, 2, false>(P, smem, m0, n0, klo, nk, acc);
  // (The same holds where the result becomes an operand: with kind 2's loop alone the 256-tile's accumulators were spilled, 3.1 ms instead of 1.1.)
  // (No batch has kinds 0 and 1 with several terms, nor as 256-tiles here, but the code that the compiler makes for kind 2 is better with them in
  // the kernel: without, two halves of 22016 x 4096 weights take 2551 us instead of 2522, and a solve with 1024 columns 977 instead of 967.)
  } else if (P.nterm > 1) {
    if (P.kind == 0) tile_loop<BT, 0, true>(P, smem, m0, n0, klo, nk, acc);
    else if (P.kind == 1) tile_loop<BT, 1, true>(P, smem, m0, n0, klo, nk, acc);
    else tile_loop<BT, 2, true>(P, smem, m0, n0, klo, nk, acc);
  } else {
    if (P.kind == 0) tile_loop<BT, 0, false>(P, smem, m0, n0, klo, nk, acc);
    else if (P.kind == 1) tile_loop<BT, 1, false>(P, smem, m0, n0, klo, nk, acc);
    else tile_loop<BT, 2, false>(P, smem, m0, n0, klo, nk, acc);
  }

  // ---- epilogue.  MFMA 32x32 result: register v of a lane holds row 8*(v/4) + 4*(lane/32) + v%4,
  // column lane%32 of the block.
  if (skipped && P.store_mode == 0) return;
  if (SPLIT && P.split > 1) {
    store_partial<BT>(P.partial + (int64_t)(part * nt + id) * (BT * BT), acc);
    return;
  }
  if (OPERAND && skipped) return;      // (the blocks below the diagonal are never read)
  wait_vm_and_lds<0>();      // (said here again, where all loops meet: else the compiler counts their loads among the tile's and waits for all of these)
  if constexpr (OPERAND) store_operand<BT>(P, m0, n0, acc);
  else store_tile<BT>(P.C, uniform(P.ldc), uniform(P.M), uniform(P.N), uniform(P.store_mode), m0, n0, acc);
}

// C[i][i] += sum_k L0[i][k]^2 over all of K, of a problem whose other sums are taken in parts or by narrow_kernel: a workgroup's first wavefront per 32
// rows, which takes the 32 x 32 block of its tile's products in the same order as a tile that is not split.  (The diagonal of H decides the order of
// the columns in act_order, by differences that are of the size of the rounding; the same sums keep the same order.)  A chain of K / 16 MFMAs whose
// one operand comes straight from memory, 40 loads ahead; it ends before the parts do.  K may be as short as 64: the loads ahead of a short
// sum stop at its last step.
__device__ __forceinline__ void diagonal_block(const GemmProblem& P, int block) {
  const int lane = threadIdx.x & 63, rl = lane & 31, row = 32 * block + rl;
  if (32 * block >= P.M) return;
  constexpr int AHEAD = 40;                // k-steps of 16
  const int steps = P.K / 16;              // (even)
  const uint16_t* src = P.term[0].L[0] + (int64_t)row * 32 + 8 * (lane >> 5);
  auto at = [&](int step) { return *reinterpret_cast<const u32x4*>(src + (int64_t)(step >> 1) * P.term[0].ktl + (step & 1) * 16); };
  u32x4 f[AHEAD];
#pragma unroll
  for (int a = 0; a < AHEAD; ++a) f[a] = at(min(a, steps - 1));
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  auto multiply = [&](const u32x4& r) {
    const bf16x8 x = __builtin_bit_cast(bf16x8, r);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, x, acc, 0, 0, 0);
  };
  int s0 = 0;
  // (a running pointer: the address of a step from its number takes longer than the step)
  const uint16_t* next = src + (AHEAD / 2) * P.term[0].ktl;
  for (; s0 + 2 * AHEAD <= steps; s0 += AHEAD)
#pragma unroll
    for (int a = 0; a < AHEAD; a += 2) {
      multiply(f[a]);
      f[a] = *reinterpret_cast<const u32x4*>(next);
      multiply(f[a + 1]);
      f[a + 1] = *reinterpret_cast<const u32x4*>(next + 16);
      next += P.term[0].ktl;
      __builtin_amdgcn_sched_barrier(0);
    }
  for (; s0 + AHEAD <= steps; s0 += AHEAD)
#pragma unroll
    for (int a = 0; a < AHEAD; ++a) {
      multiply(f[a]);
      f[a] = at(min(s0 + a + AHEAD, steps - 1));
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
  for (int a = 0; a < AHEAD; ++a)
    if (s0 + a < steps) multiply(f[a]);
#pragma unroll
  for (int v = 0; v < 16; ++v)
    if (8 * (v >> 2) + 4 * (lane >> 5) + (v & 3) == rl && row < P.M) P.C[(int64_t)row * P.ldc + row] += acc[v];
}

// CAPPED = false: one workgroup per tile.  CAPPED = true: a workgroup takes tiles blockIdx.x, blockIdx.x + gridDim.x,
// ...: the caller caps the grid to leave compute units to a kernel running beside this one.  The grid is a multiple
// of 8 then, so a workgroup's tiles all belong to its own XCD's share.
// REMAINDER: a batch of kinds 3 and 0 (a kernel of its own: in one with the other loops theirs lost 5 %).
// OPERAND: the result as an operand of another product (store_mode 3).
template <int BT, bool CAPPED, bool SPLIT = false, bool REMAINDER = false, bool OPERAND = false>
__global__ __launch_bounds__(256, BT == 128 ? 2 : 1) void gemm_nt_kernel(GemmBatch b) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if (!CAPPED) {
    if (SPLIT && (int)blockIdx.x < b.diag_wgs) { if (threadIdx.x < 64) diagonal_block(b.p[1], blockIdx.x); }
    else gemm_tile<BT, false, SPLIT, REMAINDER, OPERAND>(b, smem, blockIdx.x - (SPLIT ? b.diag_wgs : 0));
  } else {
    const int total = b.ntiles[0] + b.ntiles[1];
    for (int wid = blockIdx.x; wid < total; wid += gridDim.x) {
      gemm_tile<BT, true, false, false, false>(b, smem, wid);
      __syncthreads();                   // the last fragment reads of this tile before the next tile's loads land in LDS
    }
  }
}

// C += the sum of the parts of K, taken in their order: C is rounded once a call, as with one part (added to it one by one, the parts cost
// up to 16 roundings of a total that a series of calls has made large: error of dXXT at n = 512 after 16 calls of 8192 tokens 3.5e-7,
// 2.0e-7 so, 3.1e-7 without parts; 105 us a call of 32768 tokens either way).  grid: four workgroups (the four wavefronts of the product) per tile, problem after
// problem; a wavefront takes a 32 x 32 block.  Bound by its reads, 64 KB a tile and part.
__global__ __launch_bounds__(256) void add_parts_kernel(GemmBatch b) {
  constexpr int BT = 128, FR = 2;
  const int first = b.p[0].split > 1 ? b.ntiles[0] / b.p[0].split : 0;       // (a problem that is not split has nothing here)
  int id = blockIdx.x >> 2, pi = 0;
  if (id >= first) { id -= first; pi = 1; }
  const GemmProblem& P = b.p[pi];
  const int w = blockIdx.x & 3, blk = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int tm, tn;
  tile_position(P, id, tm, tn);
  const int row0 = tm * BT + (w >> 1) * 64 + (blk / FR) * 32 + 4 * (lane >> 5), col = tn * BT + (w & 1) * 64 + (blk % FR) * 32 + (lane & 31);
  const f32x4* src = reinterpret_cast<const f32x4*>(P.partial + (int64_t)id * (BT * BT)) + (w * (FR * FR) + blk) * 256 + lane;
  const int64_t step = (int64_t)(b.ntiles[pi] / P.split) * (BT * BT / 4);
  float c[4][4], sum[4][4];
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = row0 + 8 * v + q;
      c[v][q] = P.C[(int64_t)min(row, P.M - 1) * P.ldc + min(col, P.N - 1)];
      sum[v][q] = 0.f;
    }
  for (int s = 0; s < P.split; ++s)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const f32x4 x = src[s * step + 64 * v];
#pragma unroll
      for (int q = 0; q < 4; ++q) sum[v][q] += x[q];
    }
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (row0 + 8 * v + q < P.M && col < P.N && !(pi && b.diag_wgs && row0 + 8 * v + q == col)) P.C[(int64_t)(row0 + 8 * v + q) * P.ldc + col] = c[v][q] + sum[v][q];
}

// C += L R^T for the two problems of a batch whose tiles are few: one workgroup per 32 x 64 block of C, its eight wavefronts take an eighth
// of K each and add their sums up through LDS, in order, before C is rounded once.  So nothing but C is written, and a CU for every 128-tile
// becomes one for each of its eight blocks.  Operand fragments come straight from memory, kNarrowAhead k-tiles ahead, 8 KB a k-tile for 16
// MFMAs.  Bound by what a CU is given, some 20 bytes a clock, and by the latency in front of it: 1 MB a workgroup in 19 us at 8 columns and 4096
// tokens, two workgroups, and in 22 at 512 columns, full form, 200 of them.  H's diagonal is left to diagonal_block.
constexpr int kNarrowRows = 32, kNarrowCols = 64, kNarrowAhead = 4;
template <int NL>
__device__ __forceinline__ void narrow_loop(const GemmTerm& tm, int row0, int col0, int k0, int k1, f32x4 (&acc)[2][4]) {
  // (16 rows of a k-tile are 1 KB in a row, and one load: with 32 x 32 products a load takes half of each of twice as many lines)
  const int lane = threadIdx.x & 63, in_tile = (lane & 15) * 32 + 8 * (lane >> 4);
  const int64_t row_at = (int64_t)row0 * 32 + in_tile, col_at = (int64_t)col0 * 32 + in_tile, step = tm.ktl;
  u32x4 l[kNarrowAhead][NL][2], r[kNarrowAhead][4];
  auto load = [&](int set, int k) {
    const int64_t at = (int64_t)min(k, k1 - 1) * step;
#pragma unroll
    for (int o = 0; o < NL; ++o)
#pragma unroll
      for (int i = 0; i < 2; ++i) l[set][o][i] = *reinterpret_cast<const u32x4*>(tm.L[o] + at + row_at + 512 * i);
#pragma unroll
    for (int j = 0; j < 4; ++j) r[set][j] = *reinterpret_cast<const u32x4*>(tm.R[0] + at + col_at + 512 * j);
    __builtin_amdgcn_sched_barrier(0);
  };
  if (k1 <= k0) return;
#pragma unroll
  for (int a = 0; a < kNarrowAhead; ++a) load(a, k0 + a);
  auto multiply = [&](int a) {
#pragma unroll
    for (int o = 0; o < NL; ++o)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, l[a][o][i]), __builtin_bit_cast(bf16x8, r[a][j]), acc[i][j], 0, 0, 0);
  };
  int k = k0;                       // (no branch between the loads of a round: the compiler would wait for all of them)
  for (; k + kNarrowAhead <= k1; k += kNarrowAhead)
#pragma unroll
    for (int a = 0; a < kNarrowAhead; ++a) {
      multiply(a);
      load(a, k + a + kNarrowAhead);
    }
#pragma unroll
  for (int a = 0; a < kNarrowAhead - 1; ++a)
    if (k + a < k1) multiply(a);
}
__global__ __launch_bounds__(512, 2) void narrow_kernel(GemmBatch b) {
  __shared__ __attribute__((aligned(16))) f32x4 sums[8][8][64];          // by wavefront and piece of four rows
  if ((int)blockIdx.x < b.diag_wgs) {
    if (threadIdx.x < 64) diagonal_block(b.p[1], blockIdx.x);
    return;
  }
  int id = blockIdx.x - b.diag_wgs, pi = 0, ntile = b.ntiles[0];
  if (id >= ntile) { pi = 1; id -= ntile; ntile = b.ntiles[1]; }
  const GemmProblem& P = b.p[pi];
  {                                                                      // one run of blocks per XCD: they share their rows
    const int per = ntile >> 3, rem = ntile & 7, xcd = id & 7, loc = id >> 3;
    id = xcd < rem ? xcd * (per + 1) + loc : rem * (per + 1) + (xcd - rem) * per + loc;
  }
  int tr = 0, tc;
  if (P.tile_mode == 2) {                                                // block rows 2 t and 2 t + 1 begin at block column t
    for (int in_row = P.tiles_n; id >= in_row; ++tr) { id -= in_row; in_row = P.tiles_n - ((tr + 1) >> 1); }
    tc = (tr >> 1) + id;
  } else {
    tr = id / P.tiles_n;
    tc = id - tr * P.tiles_n;
  }
  const int row0 = uniform(tr * kNarrowRows), col0 = uniform(tc * kNarrowCols);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, nk = P.K / kGemmBK;
  f32x4 acc[2][4];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i >> 2][i & 3] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int k0 = (int)((int64_t)nk * wave / 8), k1 = (int)((int64_t)nk * (wave + 1) / 8);
  if (P.kind == 0) narrow_loop<1>(P.term[0], row0, col0, k0, k1, acc);
  else narrow_loop<2>(P.term[0], row0, col0, k0, k1, acc);
#pragma unroll
  for (int i = 0; i < 8; ++i) sums[wave][i][lane] = acc[i >> 2][i & 3];
  // wavefront w adds piece w up, 16 x 16 of C (a lane holds rows 4 (lane / 16) + 0 .. 3)
  const int row = row0 + 16 * (wave >> 2) + 4 * (lane >> 4), col = col0 + 16 * (wave & 3) + (lane & 15);
  float c[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) c[q] = P.C[(int64_t)min(row + q, P.M - 1) * P.ldc + min(col, P.N - 1)];
  __syncthreads();
  f32x4 sum = sums[0][wave][lane];
#pragma unroll
  for (int w = 1; w < 8; ++w) sum += sums[w][wave][lane];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (row + q < P.M && col < P.N && !(pi && row + q == col)) P.C[(int64_t)(row + q) * P.ldc + col] = c[q] + sum[q];
}
hipError_t launch_narrow_sums(const GemmBatch& b, hipStream_t s) {
  GemmBatch bb = b;
  if (b.nprob != 2) return hipErrorInvalidValue;
  int total = 0;
  for (int i = 0; i < 2; ++i) {
    GemmProblem& q = bb.p[i];
    if (q.kind != 1 - i || q.nterm != 1 || q.k_mode || q.store_mode || q.M != q.N || q.K <= 0 || q.K % kGemmBK || (i == 1 && q.tile_mode != 2)) return hipErrorInvalidValue;
    q.tiles_m = (q.M + kNarrowRows - 1) / kNarrowRows;
    q.tiles_n = (q.N + kNarrowCols - 1) / kNarrowCols;
    bb.ntiles[i] = 0;
    for (int r = 0; r < q.tiles_m; ++r) bb.ntiles[i] += q.tiles_n - (q.tile_mode == 2 ? r >> 1 : 0);
    total += bb.ntiles[i];
  }
  bb.diag_wgs = (bb.p[1].tiles_m + 7) / 8 * 8;                            // (a multiple of 8, which leaves the blocks on their XCDs)
  hipLaunchKernelGGL(narrow_kernel, dim3(bb.diag_wgs + total), dim3(512), 0, s, bb);
  return hipGetLastError();
}

static LdsLimitOnce g_lds256, g_lds128, g_lds256c, g_lds128c, g_lds128s, g_lds256r, g_lds128r, g_lds256o, g_lds128o;
hipError_t launch_gemm(const GemmBatch& b, hipStream_t s) {
  GemmBatch bb = b;
  int total = 0, part_tiles = 0;
  const bool remainder = b.p[0].kind == 3;
  for (int i = 0; i < 2; ++i) {
    const GemmProblem& q = bb.p[i];
    if (bb.p[i].split < 1) bb.p[i].split = 1;
    if (i < bb.nprob && q.quartered && (!remainder || bb.tile != 256 || i != 1 || q.tile_mode != 2 || q.store_mode || q.deal || q.quartered % 2)) return hipErrorInvalidValue;
    bb.ntiles[i] = i >= bb.nprob ? 0 : 3 * q.quartered + q.split * (q.tile_mode == 2 ? q.tiles_m * (q.tiles_m + 1) / 2 : q.tiles_m * q.tiles_n);
    if (q.split > 1 && (bb.tile != 128 || q.k_mode || q.store_mode || q.deal || !q.partial)) return hipErrorInvalidValue;
    if (i < bb.nprob && q.kind == 3 && (q.nterm != 1 || q.k_mode || q.K % (2 * kGemmBK) || q.K > kMaxRemainderK)) return hipErrorInvalidValue;
    if (i < bb.nprob && remainder && (q.split > 1 || b.max_wgs > 0 || (q.kind != 3 && (q.kind != 0 || q.nterm != 1)))) return hipErrorInvalidValue;
    if (i < bb.nprob && b.max_wgs > 0 && q.kind != 2) return hipErrorInvalidValue;
    if (i < bb.nprob && q.store_mode == 3 && (bb.nprob != 1 || q.kind != 2 || q.nterm != 1 || q.split > 1 || b.max_wgs > 0 || !q.out_hi || !q.out_lo)) return hipErrorInvalidValue;
    total += bb.ntiles[i];
    if (q.split > 1) part_tiles += bb.ntiles[i] / q.split;
  }
  if (total == 0) return hipSuccess;
  // (a multiple of 8, which leaves the tiles on their XCDs; the last ones may have no rows)
  bb.diag_wgs = bb.nprob == 2 && bb.p[1].split > 1 && bb.p[1].tile_mode == 2 ? (4 * bb.p[1].tiles_m + 7) / 8 * 8 : 0;
  hipError_t e = g_lds256.ensure(reinterpret_cast<const void*>(&gemm_nt_kernel<256, false>), kLds256);
  if (e == hipSuccess) e = g_lds128.ensure(reinterpret_cast<const void*>(&gemm_nt_kernel<128, false>), kLds128);
  if (e == hipSuccess) e = g_lds256c.ensure(reinterpret_cast<const void*>(&gemm_nt_kernel<256, true>), kLds256);
  if (e == hipSuccess) e = g_lds128c.ensure(reinterpret_cast<const void*>(&gemm_nt_kernel<128, true>), kLds128);
  if (e == hipSuccess) e = g_lds128s.ensure(reinterpret_cast<const void*>(&gemm_nt_kernel<128, false, true>), kLds128);
  if (e == hipSuccess) e = g_lds256r.ensure(reinterpret_cast<const void*>(&gemm_nt_kernel<256, false, false, true>), kLds256);
  if (e == hipSuccess) e = g_lds128r.ensure(reinterpret_cast<const void*>(&gemm_nt_kernel<128, false, false, true>), kLds128);
  if (e == hipSuccess) e = g_lds256o.ensure(reinterpret_cast<const void*>(&gemm_nt_kernel<256, false, false, false, true>), kLds256);
  if (e == hipSuccess) e = g_lds128o.ensure(reinterpret_cast<const void*>(&gemm_nt_kernel<128, false, false, false, true>), kLds128);
  if (e != hipSuccess) return e;
  if (b.p[0].store_mode == 3) {
    if (b.tile == 256) hipLaunchKernelGGL((gemm_nt_kernel<256, false, false, false, true>), dim3(total), dim3(256), kLds256, s, bb);
    else hipLaunchKernelGGL((gemm_nt_kernel<128, false, false, false, true>), dim3(total), dim3(256), kLds128, s, bb);
  } else if (remainder) {
    if (b.tile == 256) hipLaunchKernelGGL((gemm_nt_kernel<256, false, false, true>), dim3(total), dim3(256), kLds256, s, bb);
    else hipLaunchKernelGGL((gemm_nt_kernel<128, false, false, true>), dim3(total), dim3(256), kLds128, s, bb);
  } else if (part_tiles) {
    hipLaunchKernelGGL((gemm_nt_kernel<128, false, true>), dim3(bb.diag_wgs + total), dim3(256), kLds128, s, bb);
    hipLaunchKernelGGL(add_parts_kernel, dim3(4 * part_tiles), dim3(256), 0, s, bb);
  } else if (b.max_wgs > 0 && b.max_wgs < total) {
    const int grid = b.max_wgs >= 8 ? b.max_wgs / 8 * 8 : 8;
    if (b.tile == 256)
      hipLaunchKernelGGL((gemm_nt_kernel<256, true>), dim3(grid), dim3(256), kLds256, s, bb);
    else
      hipLaunchKernelGGL((gemm_nt_kernel<128, true>), dim3(grid), dim3(256), kLds128, s, bb);
  } else if (b.tile == 256) {
    hipLaunchKernelGGL((gemm_nt_kernel<256, false>), dim3(total), dim3(256), kLds256, s, bb);
  } else {
    hipLaunchKernelGGL((gemm_nt_kernel<128, false>), dim3(total), dim3(256), kLds128, s, bb);
  }
  return hipGetLastError();
}

}  // namespace gptaq
