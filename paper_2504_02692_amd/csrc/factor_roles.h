// The fp64 part of the factor sweep (Algorithm 1, line 3), as parts of the sweep's launches (factor_sweep.hip).  One 256-column outer
// block OB at a time:
//   factor_role   : F_OB,OB = V V^T, V upper triangular, in one workgroup;
//   panel_role    : V_I,OB = F_I,OB V_OB,OB^-T for the rows I above OB, and U_OB,OB = V_OB,OB^-1, written as the digit
//                   operands of the rank-256 products (gemm_i8s.h).
//
// All count indices of the block from its end, r -> 255 - r, which turns the factorisation "from the last column to the
// first" into the usual one: S = V V^T with V lower triangular, columns 0, 1, ... (S, V, W = V^-1 below are in this order;
// where the matrix ends the block is filled up with the identity, which then comes first and couples to nothing).
//
// A 16 x 16 tile of fp64 is held by a wavefront as lane l, register v: row l % 16, column 4 (l / 16) + v.  That is at once
// (columns c and rows of the contraction counted in the order 4 (l / 16) + v)
//   * the B operand of four v_mfma_f64_16x16x4 (contraction over the tile's columns), and
//   * their result, when the A operand's lane l carries row perm(l % 16) of its tile, perm(4 v + g) = 4 g + v,
// so  T_ab^T -= X_b X_a^T  and  X_a^T = W_k T_ak^T  chain from accumulator to operand without a shuffle.  In memory and
// LDS a tile is two runs of 64 x 16 bytes: registers 0, 1 of every lane, then 2, 3.
//
// What bounds them: one chain.  A block of 256 columns of a small matrix, in us: 2.8 until the first tiles are there, 14 for each half
// (a tile 1.7 to 1.9: 1.28 of its 16 column steps, each a reciprocal, its Newton steps and an update; 0.5 until the next diagonal tile is
// updated and handed over), about 4 between them (the last column, the rows from the other workgroups, the rest of the update and its way
// back, less the first tile's factorisation), 1.5 for the last column of the panel and 3 for its digits and their way to memory: 43 in
// all, and about 50 beside products.  As launches of their own, the factorisation in one workgroup of eight wavefronts, panel and products
// on two streams, it was 48 + 16 and 15 to 20 of events; with a launch for each half, the rows and the update between them 16 + 7 + 6 + 16.
// An f64 MFMA (64 clocks for 1024 products) is no faster than v_fma_f64, but its operands are one register a lane.
// gptaq_prepare with a copy of H and dXXT in front of it, at n = 512 / 1024 / 4096 / 11008, us: 252 / 454 / 1992 / 18222 -> 167 / 313 / 1535 / 16965.
#pragma once
#include "common.h"
#include "gemm_i8s.h"
#include "patience.h"
#include <utility>

namespace gptaq {

typedef __attribute__((ext_vector_type(2))) double f64x2;
typedef __attribute__((ext_vector_type(4))) double f64x4;

namespace {
constexpr int NT = kFactorBlock / 16;             // tiles per side of the block
constexpr int NH = NT / 2;                        // and of a half
constexpr int TILE = 256;                         // doubles of a tile

__device__ __forceinline__ f64x4 load_tile(const double* t, int lane) {
  const f64x2 a = *reinterpret_cast<const f64x2*>(t + 2 * lane), b = *reinterpret_cast<const f64x2*>(t + 128 + 2 * lane);
  return f64x4{a[0], a[1], b[0], b[1]};
}
__device__ __forceinline__ void store_tile(double* t, int lane, f64x4 x) {
  *reinterpret_cast<f64x2*>(t + 2 * lane) = f64x2{x[0], x[1]};
  *reinterpret_cast<f64x2*>(t + 128 + 2 * lane) = f64x2{x[2], x[3]};
}
// the same for a reader on another CU in the same launch: written through to where all XCDs see it (see BlockSync)
__device__ __forceinline__ void publish_tile(double* t, int lane, f64x4 x) {
#pragma unroll
  for (int v = 0; v < 4; ++v) __hip_atomic_store(t + (v >> 1) * 128 + 2 * lane + (v & 1), x[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// lane whose part of a stored tile is the A operand of lane l
__device__ __forceinline__ int operand_lane(int lane) { return (lane & 48) | (4 * (lane & 3)) | ((lane >> 2) & 3); }

// F[row][col + 3 .. col] (four columns, counted from the end), 0 past column n.  The addresses are clamped instead of predicated:
// a branch per entry would wait for every load before the next one is sent.  col % 4 == 0; ldf is a multiple of 16.
__device__ __forceinline__ f64x4 load_row4(const double* F, int64_t ldf, int n, int row, int col) {
  const double* p = F + (int64_t)min(row, n - 1) * ldf + (col < ldf ? col : 0);
  const f64x2 a = *reinterpret_cast<const f64x2*>(p), b = *reinterpret_cast<const f64x2*>(p + 2);
  return f64x4{col + 3 < n ? b[1] : 0.0, col + 2 < n ? b[0] : 0.0, col + 1 < n ? a[1] : 0.0, col < n ? a[0] : 0.0};
}

// c + (A tile) x (B tile), contraction over both tiles' 16 columns
__device__ __forceinline__ f64x4 tile_product(f64x4 a, f64x4 b, f64x4 c) {
#pragma unroll
  for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], c, 0, 0, 0);
  return c;
}

// LDS-only barrier: the stores to memory of a step need not have arrived.  The products of a step stay in front of it (the
// compiler is free to move them past, into the time of the next step's first, critical ones: 6 us of 60).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// LDS written by some lanes of a wavefront becomes readable by its others: the hardware keeps a wavefront's accesses in order,
// the compiler does behind a fence
__device__ __forceinline__ void wave_publish() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// acc += (lane C of each group of 16 lanes of s) * e.  The compiler does not look into the asm: s must not have been written by
// the two instructions before (row_value below waits; every later use is behind a chain of results of that one;
// tests/test_dpp_hazards.py checks the machine code for it).
template <int C> __device__ __forceinline__ void fmac_lane(double& acc, double s, double e) {
  asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(s), "v"(e), "n"(C));
}
template <int C> __device__ __forceinline__ double row_value(double s) {      // lane C of each group of 16 lanes
  double r;
  asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(s), "n"(C));
  return r;
}

// hardware estimate (about 26 bits) and one step of third order (about 1 ulp)
__device__ __forceinline__ double rsqrt_of(double x) {
  const double r = __builtin_amdgcn_rsq(x), e = fma(-x * r, r, 1.0);          // (1 - e)^(-1/2) = 1 + e / 2 + 3 e^2 / 8 + ...
  return fma(r * e, fma(e, 0.375, 0.5), r);
}

// ---- several workgroups of one launch work on a block: one factors it, others follow it tile column by tile column.  A workgroup
// draws a number when it starts, and the parts are dealt in the order of the numbers: the nine that factor the block and wait for one
// another come first, and a panel, which waits for these, starts when they are running, whatever the order in which the hardware starts
// them; and nobody waits for the workgroups that do products.
// What one writes for another goes past its XCD's L2 (publish_tile), and a flag behind it once the stores have been acknowledged.  The
// reader's own L2 cannot hold an older copy: nothing reads these lines earlier in the launch, and a launch starts with clean caches.
// All words are 0 before the call's first launch.
struct BlockSync {
  static constexpr int kTicket = 56, kWords = kBlockSyncBytes / 4;
  static constexpr int column(int k, int w) { return 3 * k + w; }          // W_kk and the rows of wavefront w + 1 of tile column k
  static constexpr int row(int m) { return 48 + m; }                       // tile row NH + m on the first half's columns
  static constexpr int tile(int m, int w) { return 64 + 4 * m + w; }       // tiles w, w + 4 of row m of the second half's updated block
  static constexpr int cell(int m, int k) { return 128 + 8 * m + k; }      // tile row NH + m on tile column k < NH
};
__device__ __forceinline__ void set_flag(int32_t* sync, int word, int lane) {      // (behind a wait for the stores it stands for)
  if (lane == 0) __hip_atomic_store(sync + word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <int N> __device__ __forceinline__ void wait_stores() {           // all but the last N memory accesses of the wavefront are done
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}
constexpr int kFactorTeam = 1 + NH;               // workgroups that factor a block
static_assert(GPTAQ_INFO_STALLED < -(1 + (1 << 24)), "no row's code");
struct Flags {
  int32_t* words;                                // 64 of them, one a lane
  const BlockFactor& f;
  int lane;
  uint64_t seen = 0;
  __device__ __forceinline__ bool ready(uint64_t need) const { return (seen & need) == need; }
  // Waits until the flags of `need` are set, or for as long as Patience has: then info says so.
  __device__ __forceinline__ void wait(uint64_t need) {
    Patience patience;
    while (!ready(need)) {
      seen = __ballot(__hip_atomic_load(words + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0);
      if (ready(need)) break;
      __builtin_amdgcn_s_sleep(2);
      if (patience.over([&]() { return __hip_atomic_load(f.sync + BlockSync::kTicket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= kFactorTeam; })) {
        if (lane == 0) atomicMin(f.info, GPTAQ_INFO_STALLED);
        seen = ~0ull;
      }
    }
    asm volatile("" ::: "memory");
  }
};

struct FactorShared {
  double x[NH][TILE];        // V_ak of the current tile column k
  double diag[TILE];         // tile (k, k) before its factorisation, entry (row, column) at 16 column + row
  double w[TILE];            // W_kk, as a stored tile
};

// ---- the 16 x 16 factorisation, one wavefront.  Every group of 16 lanes holds the whole symmetric tile, lane r row r in
// registers s[0..15]; a step needs the pivot column in every lane, and by symmetry lane c's s[j] is S[c][j]: a broadcast inside
// the group of 16 (DPP) delivers it as an operand of the product.  f: rows of the identity taken through the same steps, which
// makes them the rows of V^-T.
// The updates of step J, s[J+1..15] and then f[J+1..15], in one list: all but the first are independent work for the time the
// next pivot's broadcast and reciprocal take (the compiler's own order left a third of the chain uncovered).
template <int J, int FROM, int TO>
__device__ __forceinline__ void step_updates(double (&s)[16], double (&f)[16], double ns, double nf) {
  constexpr int N = 2 * (15 - J), END = TO < N ? TO : N;
  if constexpr (FROM < END) {
    constexpr int C = FROM < 15 - J ? J + 1 + FROM : 2 * J - 14 + FROM;
    if constexpr (FROM < 15 - J) fmac_lane<C>(s[C], s[J], ns); else fmac_lane<C>(f[C], s[J], nf);
    step_updates<J, FROM + 1, TO>(s, f, ns, nf);
  }
}
// q: 1 / pivot J, or 0 if that is not positive
template <int J>
__device__ __forceinline__ void factor_steps(double (&s)[16], double (&f)[16], double& piv, double q, int r) {
  if constexpr (J < 15) {
    const double ns = -(s[J] * q);
    step_updates<J, 0, 1>(s, f, ns, 0.0);
    __builtin_amdgcn_sched_barrier(0);
    const double nf = -(f[J] * q);
    step_updates<J, 1, 3>(s, f, ns, nf);
    __builtin_amdgcn_sched_barrier(0);
    const double p = row_value<J + 1>(s[J + 1]);
    __builtin_amdgcn_sched_barrier(0);
    step_updates<J, 3, 5>(s, f, ns, nf);
    __builtin_amdgcn_sched_barrier(0);
    const double x = __builtin_amdgcn_rcp(p);
    __builtin_amdgcn_sched_barrier(0);
    piv = r == J + 1 ? p : piv;
    step_updates<J, 5, 8>(s, f, ns, nf);
    const double x0 = p > 0.0 ? x : 0.0;
    __builtin_amdgcn_sched_barrier(0);
    const double e = fma(-p, x0, 1.0);
    __builtin_amdgcn_sched_barrier(0);
    step_updates<J, 8, 9>(s, f, ns, nf);
    __builtin_amdgcn_sched_barrier(0);
    const double e2 = fma(e, e, e);
    __builtin_amdgcn_sched_barrier(0);
    step_updates<J, 9, 10>(s, f, ns, nf);
    __builtin_amdgcn_sched_barrier(0);
    const double qn = fma(e2, x0, x0);           // the estimate's 26 bits and one step of third order: about 1 ulp
    step_updates<J, 10, 32>(s, f, ns, nf);
    factor_steps<J + 1>(s, f, piv, qn, r);
  }
}

// w[c] = f[c] * (lane c of each group of 16 lanes of s)
template <int... C>
__device__ __forceinline__ void scale_by_lane(double (&w)[16], double s, const double (&f)[16], std::integer_sequence<int, C...>) {
  ((w[C] = 0.0, fmac_lane<C>(w[C], s, f[C])), ...);
}

__device__ __forceinline__ void factor_diag(FactorShared& sh, int32_t* info, int last_index) {
  const int lane = threadIdx.x & 63, r = lane & 15;
  double s[16], f[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    s[c] = sh.diag[16 * c + r];
    f[c] = c == r ? 1.0 : 0.0;
  }
  double piv = row_value<0>(s[0]);                            // of lane r: pivot r, once its step is reached
  const double x0 = piv > 0.0 ? __builtin_amdgcn_rcp(piv) : 0.0, e = fma(-piv, x0, 1.0);
  factor_steps<0>(s, f, piv, fma(fma(e, e, e), x0, x0), r);
  const uint64_t bad = __ballot(!(piv > 0.0)) & 0xffff;       // the first pivot in the order of the factorisation is reported
  if (bad && lane == 0) atomicCAS(info, 0, last_index - __builtin_ctzll(bad));
  // column c of V and row c of W are scaled by 1 / sqrt(pivot c)
  double rs = piv > 0.0 ? rsqrt_of(piv) : 1.0;
  asm volatile("s_nop 1" : "+v"(rs));
  double w[16];
  scale_by_lane(w, rs, f, std::make_integer_sequence<int, 16>{});
  // w[c] of lane i is W[c][i]: tile position of (row c, column i)
  if (lane < 16) {
    double* dst = sh.w + (((r >> 1) & 1) * 128 + (r >> 2) * 32 + (r & 1));
#pragma unroll
    for (int c = 0; c < 16; ++c) dst[2 * c] = w[c];
  }
}

// entry block (a, b) of OB, a >= b, as a tile: both halves of a diagonal one from the upper triangle of F, the identity past column n
__device__ __forceinline__ f64x4 load_block_tile(const BlockFactor& a, int ta, int tb, int r, int g) {
  const int last = a.o0 + kFactorBlock - 1, row = 16 * ta + r;
  if (tb < ta) return load_row4(a.F, a.ldf, a.n, last - row, last - 3 - 16 * tb - 4 * g);
  f64x4 d;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int col = 16 * tb + 4 * g + v, fi = last - max(row, col), fj = last - min(row, col);
    const double x = a.F[(int64_t)min(fi, a.n - 1) * a.ldf + min(fj, a.n - 1)];
    d[v] = fj < a.n ? x : (fi == fj ? 1.0 : 0.0);
  }
  return d;
}
// tile (a, b) of the second half's own block after the first half's update, a >= b
__device__ __forceinline__ double* half_tile(const BlockFactor& a, int ta, int tb) { return a.T + (ta * (ta + 1) / 2 + tb) * TILE; }
__device__ __forceinline__ double* factor_tile(double* V, int k, int a) { return V + ((int64_t)k * NT + a) * TILE; }

// ---- the block's factorisation, one workgroup, a half after the other.  Wavefront 0 factors the diagonal tiles; the other three hold
// the tiles (a, 0 .. a) of these rows a of the half in registers from load to end, about as many products each:
__host__ __device__ constexpr int tile_row(int w, int i) {
  constexpr int8_t rows[4][3] = {{-1, -1, -1}, {7, 1, 0}, {6, 3, -1}, {5, 4, 2}};
  return rows[w][i];
}
__host__ __device__ constexpr int tile_rows(int w) { int n = 0; while (n < 3 && tile_row(w, n) >= 0) ++n; return n; }
__host__ __device__ constexpr int tile_base(int w, int i) { int b = 0; for (int q = 0; q < i; ++q) b += tile_row(w, q) + 1; return b; }

template <int W, int HALF>
__device__ __forceinline__ void factor_rows(const BlockFactor& a, FactorShared& sh) {
  constexpr int NR = tile_rows(W), first = NH * HALF;
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4, ol = operand_lane(lane);
  f64x4 t[tile_base(W, NR)];
  auto put_diag = [&](const f64x4& d) {
#pragma unroll
    for (int v = 0; v < 4; ++v) sh.diag[16 * (4 * g + v) + r] = d[v];
  };
  // The second half's first tile is there before its others (half_row_role), and its factorisation takes the time in which they come.
  Flags f{a.sync + 64, a, lane};
  if (HALF) {
    if (W == 1) {
      f.wait(1ull);
      put_diag(load_tile(half_tile(a, 0, 0), lane));
    }
    lds_barrier();
    f.wait(0xffffffffull);
  }
#pragma unroll
  for (int b = 0; b < NH; ++b) {                               // (in the order in which they are needed)
#pragma unroll
    for (int i = NR - 1; i >= 0; --i)
      if (b <= tile_row(W, i) && (!HALF || tile_row(W, i) > 0))
        t[tile_base(W, i) + b] = HALF ? load_tile(half_tile(a, tile_row(W, i), b), lane) : load_block_tile(a, tile_row(W, i), b, r, g);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (!HALF) {
#pragma unroll
    for (int i = 0; i < NR; ++i)
      if (tile_row(W, i) == 0) put_diag(t[tile_base(W, i)]);
    lds_barrier();
  }
#pragma clang loop unroll(full)
  for (int k = 0; k < NH; ++k) {
    lds_barrier();                                             // W_kk is in LDS; every wavefront is done with column k - 1
    if (W == 1) publish_tile(factor_tile(a.V, first + k, first + k), lane, load_tile(sh.w, lane));
    if (k == NH - 1) break;
    f64x4 nx[NR];
    const f64x4 wk = load_tile(sh.w, ol);
    auto column = [&](int i) {                                 // V_ak of the wavefront's i-th row
      const f64x4 x = tile_product(wk, t[tile_base(W, i) + k], f64x4{0.0, 0.0, 0.0, 0.0});
      store_tile(sh.x[tile_row(W, i)], lane, x);
      publish_tile(factor_tile(a.V, first + k, first + tile_row(W, i)), lane, x);
      nx[i] = -x;
    };
    // the diagonal tile that the next factorisation waits for comes first
    bool own = false;
#pragma unroll
    for (int i = 0; i < NR; ++i)
      if (tile_row(W, i) == k + 1) {
        own = true;
        __builtin_amdgcn_s_setprio(2);
        column(i);
        wave_publish();
        f64x4& d = t[tile_base(W, i) + k + 1];
        d = tile_product(load_tile(sh.x[k + 1], ol), nx[i], d);
        put_diag(d);
        __builtin_amdgcn_s_setprio(0);
      }
    // the stores of column k - 1 are a step old and have arrived
    if (k > 0) {
      if (W == 1) { if (own) wait_stores<8>(); else wait_stores<4>(); }
      else if (own) wait_stores<4>();
      else wait_stores<0>();
      set_flag(a.sync, BlockSync::column(first + k - 1, W - 1), lane);
    }
#pragma unroll
    for (int i = 0; i < NR; ++i)
      if (tile_row(W, i) > k + 1) column(i);
    lds_barrier();                                             // column k of V and the next diagonal tile are in LDS
#pragma unroll
    for (int b = k + 1; b < NH; ++b) {
      if (b > tile_row(W, 0)) continue;
      const f64x4 xb = load_tile(sh.x[b], ol);
#pragma unroll
      for (int i = 0; i < NR; ++i)
        if (tile_row(W, i) >= b && tile_row(W, i) > k + 1) {
          f64x4& d = t[tile_base(W, i) + b];
          d = tile_product(xb, nx[i], d);
        }
    }
  }
  wait_stores<0>();
  set_flag(a.sync, BlockSync::column(first + NH - 2, W - 1), lane);
  set_flag(a.sync, BlockSync::column(first + NH - 1, W - 1), lane);
}

template <int HALF>
__device__ __forceinline__ void factor_diagonal(const BlockFactor& a, FactorShared& sh) {
  lds_barrier();                                               // the first diagonal tile is in LDS
  for (int k = 0; k < NH; ++k) {
    factor_diag(sh, a.info, a.o0 + kFactorBlock - 16 * (NH * HALF + k));
    lds_barrier();
    if (k == NH - 1) break;
    lds_barrier();
  }
}

__device__ __forceinline__ void factor_role(const BlockFactor& a, FactorShared& sh) {
  switch (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {
    case 0: __builtin_amdgcn_s_setprio(3); factor_diagonal<0>(a, sh); factor_diagonal<1>(a, sh); break;
    case 1: factor_rows<1, 0>(a, sh); factor_rows<1, 1>(a, sh); break;
    case 2: factor_rows<2, 0>(a, sh); factor_rows<2, 1>(a, sh); break;
    default: factor_rows<3, 0>(a, sh); factor_rows<3, 1>(a, sh); break;
  }
}

// ---- a panel: 16 rows, one workgroup; wavefront w holds tile columns w, w + 4, ...
// Step k: their owner turns tile column k into V_ik = F_ik W_kk^T and publishes it in LDS; all update their later columns.
struct PanelShared {
  double x[2][TILE];
  double rowmax[4][16];
};
// The left operands (W_kk for its owner, V_bk of the wavefront's later columns b) are fetched a step ahead if they are there.
// after(k, V_ik negated): called by every wavefront at the end of each step but the last.
template <int STEPS, class After>
__device__ __forceinline__ void panel_steps(const double* V, f64x4 (&t)[STEPS / 4], int wave, int lane, PanelShared& sh, Flags& flags, After after) {
  constexpr int NQ = STEPS / 4;
  const int ol = operand_lane(lane);
  auto tile_of = [&](int k, int b) { return V + ((int64_t)k * NT + b) * TILE; };
  auto need = [&](int k) { return 7ull << (3 * k) | (STEPS == NT ? 0xffull << BlockSync::row(0) : 0ull); };
  f64x4 wk[2], vb[2][NQ];
  auto fetch = [&](int k) {
    if (wave == (k & 3)) wk[k & 1] = load_tile(tile_of(k, k), ol);
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      if (4 * q + 3 > k) vb[k & 1][q] = load_tile(tile_of(k, max(wave + 4 * q, k)), ol);
  };
  bool have = false;
#pragma clang loop unroll(full)
  for (int k = 0; k < STEPS; ++k) {
    if (!have) {
      flags.wait(need(k));
      fetch(k);
    }
    have = k + 1 < STEPS && flags.ready(need(k + 1));
    if (have) fetch(k + 1);
    const int q0 = k >> 2;
    if (wave == (k & 3)) {
      t[q0] = tile_product(wk[k & 1], t[q0], f64x4{0.0, 0.0, 0.0, 0.0});
      store_tile(sh.x[k & 1], lane, -t[q0]);
    }
    if (k == STEPS - 1) break;
    lds_barrier();
    const f64x4 nx = load_tile(sh.x[k & 1], lane);
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      if (4 * q + 3 > k && wave + 4 * q > k) t[q] = tile_product(vb[k & 1][q], nx, t[q]);
    after(k, nx);
  }
}

// Tile row m of OB's second half: V on the first half's columns, then the row's part of the second half's own block less the product
// of these rows.
__device__ __forceinline__ void half_row_role(const BlockFactor& a, int m, PanelShared& sh) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, g = lane >> 4, ol = operand_lane(lane);
  f64x4 x[NH / 4], t[2];
#pragma unroll
  for (int q = 0; q < NH / 4; ++q) x[q] = load_block_tile(a, NH + m, wave + 4 * q, r, g);
#pragma unroll
  for (int q = 0; q < 2; ++q) t[q] = load_block_tile(a, NH + m, NH + min(wave + 4 * q, m), r, g);
  Flags flags{a.sync, a, lane};
  // The update follows the columns, three steps behind: a row publishes a column at its step, its flag a step later, its rows are fetched by the
  // others in the step after that and multiplied in the next.  What is left behind the last column is a product of three.
  // (Row 0's one tile, which the factorisation goes on with first, needs nothing of other rows: wavefront 0 updates it from LDS, at once.)
  Flags cells{a.sync + BlockSync::cell(0, 0), a, lane};
  const uint64_t rows = m == NH - 1 ? ~0ull : (1ull << (8 * (m + 1))) - 1;
  f64x4 nx[NH], xb[3][2];
  auto fetch = [&](int k, int set) {
#pragma unroll
    for (int q = 0; q < 2; ++q) xb[set][q] = load_tile(factor_tile(a.V, k, NH + min(wave + 4 * q, m)), ol);
  };
  auto apply = [&](int k, int set) {
#pragma unroll
    for (int q = 0; q < 2; ++q) t[q] = tile_product(xb[set][q], nx[k], t[q]);
  };
  auto after = [&](int k, const f64x4& negated) {
    nx[k] = negated;
    if (wave == (k & 3)) publish_tile(factor_tile(a.V, k, NH + m), lane, x[k >> 2]);
    if (m == 0) {
      if (wave == 0) t[0] = tile_product(-load_tile(sh.x[k & 1], ol), negated, t[0]);
    } else {
      if (k >= 3) apply(k - 3, (k - 3) & 1);
      if (k >= 2) {
        cells.wait(rows & 0x0101010101010101ull << (k - 2));
        fetch(k - 2, k & 1);
      }
    }
    if (k > 0 && wave == ((k - 1) & 3)) {
      wait_stores<0>();
      set_flag(a.sync, BlockSync::cell(m, k - 1), lane);
    }
  };
  panel_steps<NH>(a.V, x, wave, lane, sh, flags, after);
  if (wave == 3) publish_tile(factor_tile(a.V, NH - 1, NH + m), lane, x[1]);
  lds_barrier();
  nx[NH - 1] = load_tile(sh.x[(NH - 1) & 1], lane);
  if (m == 0 && wave == 0) {
    t[0] = tile_product(-load_tile(sh.x[(NH - 1) & 1], ol), nx[NH - 1], t[0]);
    publish_tile(half_tile(a, 0, 0), lane, t[0]);
  }
  wait_stores<0>();
  if (m == 0) set_flag(a.sync, BlockSync::tile(0, wave), lane);
  if (wave >= 2) set_flag(a.sync, BlockSync::cell(m, wave + 4), lane);
  lds_barrier();
  if (wave == 0) set_flag(a.sync, BlockSync::row(m), lane);
  if (m == 0) return;
  apply(NH - 4, (NH - 4) & 1);
  cells.wait(rows & 0xe0e0e0e0e0e0e0e0ull);
#pragma unroll
  for (int k = NH - 3; k < NH; ++k) fetch(k, k - (NH - 3));
#pragma unroll
  for (int k = NH - 3; k < NH; ++k) apply(k, k - (NH - 3));
#pragma unroll
  for (int q = 0; q < 2; ++q)
    if (wave + 4 * q <= m) publish_tile(half_tile(a, m, wave + 4 * q), lane, t[q]);
  wait_stores<0>();
  set_flag(a.sync, BlockSync::tile(m, wave), lane);
}

// The rows above the block, and the inverse: workgroups 0 .. 15 take 16 rows of the identity through the same steps, which makes
// them rows of V^-T, i.e. columns of U_OB,OB.  The digit operands keep the matrix's own order of columns: k = 255 - (column counted
// from the end).
__device__ __forceinline__ void panel_role(const BlockFactor& f, const BlockPanel& a, int wg, PanelShared& sh) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, g = lane >> 4;
  const bool inverse = wg < NT;
  const int row0 = inverse ? 16 * wg : 16 * (wg - NT);
  f64x4 t[4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int col = 16 * (wave + 4 * q) + 4 * g + v;
      t[q][v] = col == row0 + r ? 1.0 : 0.0;
    }
  if (!inverse) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      t[q] = load_row4(f.F, f.ldf, f.n, row0 + r, f.o0 + kFactorBlock - 4 - 16 * (wave + 4 * q) - 4 * g);
  }
  Flags flags{f.sync, f, lane};
  // (U's own entries go to memory as the columns come: all of them behind the last one took 1.3 us more)
  const int j = kFactorBlock - 1 - (row0 + r);
  auto store_u = [&](int q) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = kFactorBlock - 1 - (16 * (wave + 4 * q) + 4 * g + v);
      a.Uob[j * kFactorBlock + i] = t[q][v];
      if (i <= j && f.o0 + j < f.n) a.Uout[(int64_t)i * f.ldf + j] = t[q][v];
    }
  };
  panel_steps<NT>(f.V, t, wave, lane, sh, flags, [&](int k, const f64x4&) {
    if (inverse && wave == (k & 3)) store_u(k >> 2);
  });
  // ---- digits: one scale per row, the row's 256 entries are in the four wavefronts
  double mx = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) mx = fmax(mx, fabs(t[q][v]));
  mx = fmax(mx, __shfl_xor(mx, 16, 64));
  mx = fmax(mx, __shfl_xor(mx, 32, 64));
  if (lane < 16) sh.rowmax[wave][lane] = mx;
  lds_barrier();
#pragma unroll
  for (int q = 0; q < 4; ++q) mx = fmax(mx, sh.rowmax[q][r]);
  const int e = digit_exponent(mx);
  const double sc = digit_scale(e);
  const I8Operand& o = inverse ? a.Ucol : a.Vs;
  const int row = inverse ? kFactorBlock - 1 - (row0 + r) : row0 + r;      // row of the operand
  if (wave == 0 && g == 0) o.scale[row] = e - 26;
  const int line = (row >> 3) & 3;
  uint8_t* slab = o.planes + (int64_t)(row >> 5) * 1024 + 256 * line;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    uint32_t w[kI8Planes];
    pack_digits(digits_of(t[q][3], sc), digits_of(t[q][2], sc), digits_of(t[q][1], sc), digits_of(t[q][0], sc), w);
    const int k0 = kFactorBlock - 4 - (16 * (wave + 4 * q) + 4 * g);       // k of the last of the lane's four columns
    const int slot = ((row & 7) << 1) | (((k0 >> 4) & 1) ^ (line & 1));
    uint8_t* dst = slab + (int64_t)(k0 >> 5) * o.chunk_stride() + slot * 16 + (k0 & 15);
#pragma unroll
    for (int i = 0; i < kI8Planes; ++i) *reinterpret_cast<uint32_t*>(dst + (int64_t)i * o.plane_stride()) = w[i];
  }
  if (inverse && wave == 3) store_u(NT / 4 - 1);
}
}  // namespace
}  // namespace gptaq
