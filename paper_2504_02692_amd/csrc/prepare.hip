// Algorithm 1, lines 3-4: damping, the inverse-Cholesky factor and the fused matrix P.
//
// Step 3 of the paper needs L with (H + lambda I)^-1 = L L^T.  Instead of inverting and then
// factoring, factor  H + lambda I = V V^T  with V UPPER triangular (a Cholesky factorisation
// run from the last row/column towards the first); then U = L^T = V^-1 (the factor is unique
// for a positive diagonal).  Factorisation and triangular inverse are swept together from the
// bottom-right to the top-left, in fp64, inside one n x n fp64 array F whose strictly-upper
// region holds Schur-complement data until its block column is factored and the running
// right-hand side R of the solve V U = I afterwards:
//
//   for every outer block OB of 256 columns, last to first      (I: rows above OB, J: columns right of OB)
//     factor : F_OB,OB = V_OB,OB V_OB,OB^T             one workgroup          } fp64 (block_factor.hip)
//     panel  : V_I,OB = F_I,OB V_OB,OB^-T and U_OB,OB = V_OB,OB^-1, as digits }
//     syrk   : F_II  -= V_I,OB V_I,OB^T                (rank 256)  } the n^3 * 2/3 bulk: digit-sliced operands,
//     rowblk : U_OB,J  = U_OB,OB R_OB,J                            } exact int8 MFMA products,
//     rupd   : R_I,J  -= V_I,OB U_OB,J                 (rank 256)  } fp64 recombination (gemm_i8s.hip)
//     close  : R_I,OB  = -V_I,OB U_OB,OB
//
// Theorem 4.2's two products then run on the bf16 MFMA GEMM with fp32 operands split into
// bf16 hi+lo (three cross products per term).
#include "common.h"
#include <mutex>
#include <vector>

namespace gptaq {

constexpr int NBO = kFactorBlock;             // outer block (columns per rank-256 update)

// ----------------------------------------------------------------------------- statistics
// One workgroup: dead inputs, lambda = damp * mean(diag), info words.
__global__ __launch_bounds__(1024) void diag_stats_kernel(const float* H, int64_t ldh, int n, float damp,
                                                          uint8_t* dead, double* lam_out, int32_t* info) {
  __shared__ double ssum[1024];
  __shared__ int scnt[1024];
  double s = 0.0;
  int c = 0;
  for (int i = threadIdx.x; i < n; i += 1024) {
    float d = H[(int64_t)i * ldh + i];
    const bool dd = d == 0.f;
    if (dd) { d = 1.f; ++c; }
    if (dead) dead[i] = dd ? 1 : 0;
    s += (double)d;
  }
  ssum[threadIdx.x] = s;
  scnt[threadIdx.x] = c;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) { ssum[threadIdx.x] += ssum[threadIdx.x + o]; scnt[threadIdx.x] += scnt[threadIdx.x + o]; }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *lam_out = (double)damp * ssum[0] / (double)n;
    info[0] = 0;
    info[1] = scnt[0];
  }
}

// F (upper triangle, fp64) = H + lambda I with the dead-input rule applied.
// A NaN or Inf in the upper triangle of H is reported as info[0] = -(1 + row of the entry) (smallest row wins).
__global__ void build_F_kernel(const float* H, int64_t ldh, int n, const double* lam, double* F, int64_t ldf, int32_t* info) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x, i = blockIdx.y;
  if (j >= n || j < i) return;
  const float h = H[(int64_t)i * ldh + j];
  if (!__builtin_isfinite(h)) atomicMin(info, -(1 + i));
  double v = (double)h;
  if (i == j) { if (v == 0.0) v = 1.0; v += *lam; }
  F[(int64_t)i * ldf + j] = v;
}

// --------------------------------------------------------------- extraction and splits
__device__ __forceinline__ uint16_t bf16_rne(float f) {
  __bf16 b = (__bf16)f;
  return __builtin_bit_cast(uint16_t, b);
}
__device__ __forceinline__ float bf16_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// The two products of Theorem 4.2 only read the operand blocks of kSplitBlock^2 on and above the diagonal (their tiles start
// and their k ranges begin at multiples of a tile edge that divides it), so the others are not written: a third of
// extract_U_kernel's bytes and two thirds of split_rows_kernel's.
constexpr int kSplitBlock = 256;
// The operands are k-tile-major: a tile's rows of 32 k are one run, not 64 bytes of every row (whose stride is a power of two at
// n = 4096): 147 -> 118 us per product at n = 4096, 1.32 -> 1.10 ms at n = 11008.
__device__ __forceinline__ int64_t operand_at(int64_t row, int64_t k, int64_t np) { return (k >> 5) * np * 32 + row * 32 + (k & 31); }

// U (fp32, upper, zeros below) from F; its bf16 hi/lo split row-major (Uh, Ul) and
// transposed (Uth, Utl), zero-padded to np x np.   grid (np/64, np/64), 256 threads.
__global__ __launch_bounds__(256) void extract_U_kernel(const double* F, int64_t ldf, int n, float* U, int64_t ldu,
                                                        uint16_t* Uh, uint16_t* Ul, uint16_t* Uth, uint16_t* Utl,
                                                        int64_t np) {
  __shared__ uint16_t th[64][66], tl[64][66];
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  const int c = threadIdx.x & 63, rb = threadIdx.x >> 6;
  if (c0 / kSplitBlock < r0 / kSplitBlock) {
    for (int p = 0; p < 16; ++p) {
      const int gr = r0 + rb + 4 * p, gc = c0 + c;
      if (gr < n && gc < n) U[(int64_t)gr * ldu + gc] = 0.f;
    }
    return;
  }
#pragma unroll 4
  for (int p = 0; p < 16; ++p) {
    const int r = rb + 4 * p, gr = r0 + r, gc = c0 + c;
    float u = 0.f;
    if (gr < n && gc < n) {
      if (gc >= gr) u = (float)F[(int64_t)gr * ldf + gc];
      U[(int64_t)gr * ldu + gc] = u;
    }
    const uint16_t h = bf16_rne(u);
    const uint16_t l = bf16_rne(u - bf16_f32(h));
    const int64_t o = operand_at(gr, gc, np);
    Uh[o] = h;
    Ul[o] = l;
    th[r][c] = h;
    tl[r][c] = l;
  }
  __syncthreads();
  for (int p = 0; p < 16; ++p) {
    const int r = rb + 4 * p;            // r: column of U inside the tile, c: row of U
    const int64_t o = operand_at(c0 + r, r0 + c, np);
    Uth[o] = th[c][r];
    Utl[o] = tl[c][r];
  }
}

// bf16 hi/lo split of the strictly upper triangle of an fp32 matrix (rows flagged in `zero_rows` read as 0), padded
// to np x np; entries on and below the diagonal are not read and come out as 0.  Both uses want exactly that: Eq. 17
// masks dXXT L to its strictly upper part and L is lower triangular, so entry (i, k) of dXXT only ever meets a
// non-zero of L when k > i, and the masked product itself is strictly upper.
// `info` (may be NULL): a NaN or Inf among the entries read is reported as info[0] = -(1 + row of the entry).
__global__ __launch_bounds__(256) void split_rows_kernel(const float* A, int64_t lda, int n, const uint8_t* zero_rows,
                                                         uint16_t* Ah, uint16_t* Al, int64_t np, int32_t* info) {
  const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x, r0 = 4 * (int64_t)blockIdx.y;      // four rows: 256 bytes of a k-tile
  if (c >= np || c / kSplitBlock < r0 / kSplitBlock) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t r = r0 + i, o = operand_at(r, c, np);
    float v = 0.f;
    if (r < n && c < n && c > r && !(zero_rows && zero_rows[r])) v = A[r * lda + c];
    if (info && !__builtin_isfinite(v)) atomicMin(info, -(1 + (int)r));
    const uint16_t h = bf16_rne(v);
    Ah[o] = h;
    Al[o] = bf16_rne(v - bf16_f32(h));
  }
}

}  // namespace gptaq

using namespace gptaq;

namespace {
struct PrepLayout {
  int64_t np;
  int64_t rp;                      // rows of a sliced operand that spans the whole matrix
  size_t off_F, off_lam, off_dead, off_O, off_b[6], off_Uob[2], off_V, off_pl[6], off_sc[6], total;
};
PrepLayout prep_layout(int64_t n) {
  PrepLayout L;
  const int tile = gemm_tile_for(n, n);
  L.np = round_up(n, tile);
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t r = o; o += (bytes + 255) / 256 * 256; return r; };
  L.off_lam = take(256);
  L.off_F = take((size_t)n * round_up(n, 16) * 8);
  L.off_dead = take((size_t)n);
  L.off_O = take((size_t)L.np * L.np * 4);
  for (int i = 0; i < 6; ++i) L.off_b[i] = take((size_t)L.np * L.np * 2);
  for (int i = 0; i < 2; ++i) L.off_Uob[i] = take((size_t)NBO * NBO * 8);
  L.off_V = take(kFactorTileBytes);
  // sliced operands of the rank-256 products: V_I,OB (two: the helper stream reads one while the next is
  // written), R_OB,J / U_OB,J, and U_OB,OB by columns (two) and by rows
  L.rp = round_up(n, 128);
  for (int i = 0; i < 6; ++i) {
    const int64_t rows = i < 3 ? L.rp : NBO;
    L.off_pl[i] = take(I8Operand::plane_bytes(rows));
    L.off_sc[i] = take((size_t)rows * 4);
  }
  L.total = o;
  return L;
}

}  // namespace

extern "C" size_t gptaq_prepare_workspace_bytes(int64_t n) {
  if (n <= 0) return 0;
  return prep_layout(n).total;
}

extern "C" int gptaq_prepare(float* H, float* dXXT, int64_t n, int64_t ldh, float damp, uint8_t* dead,
                             int32_t* info, void* ws, size_t ws_bytes, void* stream) {
  if (!H || !dXXT || !info || !ws) return GPTAQ_ENULL;
  // (several kernels put a row index in gridDim.y, which ends at 65535: rows of the padded n x n buffers)
  if (n <= 0 || ldh < n || n > 65280 || !(damp >= 0.f)) return GPTAQ_EDIM;
  if ((uintptr_t)ws & 255) return GPTAQ_EWORKSPACE;
  const PrepLayout L = prep_layout(n);
  if (ws_bytes < L.total) return GPTAQ_EWORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  unsigned char* base = (unsigned char*)ws;
  double* lam = (double*)(base + L.off_lam);
  double* F = (double*)(base + L.off_F);
  uint8_t* deadbuf = dead ? dead : (uint8_t*)(base + L.off_dead);
  float* Obuf = (float*)(base + L.off_O);
  I8Operand sl[6];
  for (int i = 0; i < 6; ++i) sl[i] = I8Operand{base + L.off_pl[i], (int32_t*)(base + L.off_sc[i]), i < 3 ? L.rp : (int64_t)NBO};
  const I8Operand &RJs = sl[2], &Urow = sl[5];
  const int64_t ldf = round_up(n, 16);
  uint16_t* bb[6];
  for (int i = 0; i < 6; ++i) bb[i] = (uint16_t*)(base + L.off_b[i]);
  const int64_t np = L.np;
  uint16_t *Uh = bb[0], *Ul = bb[1], *Uth = bb[2], *Utl = bb[3], *Ah = bb[4], *Al = bb[5];
  const int ni = (int)n;

  hipLaunchKernelGGL(diag_stats_kernel, dim3(1), dim3(1024), 0, s, H, ldh, ni, damp, deadbuf, lam, info);
  GPTAQ_LAUNCH_CHECK();
  hipLaunchKernelGGL(build_F_kernel, dim3((unsigned)((n + 255) / 256), (unsigned)n), dim3(256), 0, s, H, ldh, ni,
                     lam, F, ldf, info);
  GPTAQ_LAUNCH_CHECK();

  // The sweep is two chains of kernels over the outer blocks OB = nob-1 .. 0 (I: rows above, J: columns right):
  //   factor chain (caller's stream): factorisation of block column OB, digits of V_I,OB and of U_OB,OB, Schur update
  //                                   of the next block column;
  //   inverse chain (helper stream):  Schur update of the rest of F_II, then U_OB,J = U_OB,OB R_OB,J,
  //                                   R_I,J -= V_I,OB U_OB,J, R_I,OB = -V_I,OB U_OB,OB.
  // The rank-256 products run on the int8 matrix cores from digit-sliced operands (gemm_i8s.hip).
  // The inverse chain of a block needs that block's V_I,OB and U_OB,OB and nothing later from the
  // factor chain, and it only writes columns >= o0 of F while the factor chain has moved on to columns < o0,
  // so the two overlap: the small sequential kernels of one hide behind the rank-256 products of the other.
  // What it reads alternates between two sets of buffers; an event per block and direction orders the streams.
  std::lock_guard<std::mutex> side_lock(side_stream_mutex());
  const int nob = (int)((n + NBO - 1) / NBO);
  SideStream* side = side_stream(3 * nob + 2);
  if (!side) { set_last_hip_error(hipGetLastError()); return GPTAQ_ELAUNCH; }
  hipStream_t sb = side->stream;
  {
    ProfScope sweep_scope(kProfFactor, s);
    bool ok = true;
    auto chk = [&](hipError_t e) { if (e != hipSuccess && ok) { ok = false; set_last_hip_error(e); } };
    hipEvent_t ev_fork = side->events[3 * nob];
    chk(hipEventRecord(ev_fork, s));                          // the helper stream starts behind build_F
    chk(hipStreamWaitEvent(sb, ev_fork, 0));
    // dXXT (dead rows zeroed) split for the products at the end: it depends on nothing here and runs beside the first block
    hipLaunchKernelGGL(split_rows_kernel, dim3((unsigned)((np + 255) / 256), (unsigned)(np / 4)), dim3(256), 0, sb, dXXT, ldh, ni,
                       deadbuf, Ah, Al, np, info);
    chk(hipGetLastError());
    for (int ob = nob - 1; ob >= 0 && ok; --ob) {
      const int o0 = ob * NBO, o1 = (int)(n < o0 + NBO ? n : o0 + NBO), wo = o1 - o0;
      const I8Operand &Vs = sl[ob & 1], &Ucol = sl[3 + (ob & 1)];
      double* Uob = (double*)(base + L.off_Uob[ob & 1]);
      hipEvent_t ev_factored = side->events[2 * ob], ev_inverted = side->events[2 * ob + 1];
      // ---- factor chain
      double* V = (double*)(base + L.off_V);
      chk(launch_block_factor(BlockFactor{F, ldf, ni, o0, info, V}, s));
      // the digit buffers of this block were last read by the inverse chain of block ob + 2
      if (ob + 2 <= nob - 1) chk(hipStreamWaitEvent(s, side->events[2 * (ob + 2) + 1], 0));
      chk(launch_block_panel(BlockPanel{F, ldf, ni, o0, V, Vs, Ucol, Uob}, s));
      chk(hipEventRecord(ev_factored, s));
      // Schur complement of everything above/left of the outer block, F_II -= V_I,OB V_I,OB^T, in two parts:
      // the block column the next outer block factors (here, it is on the critical path) and the rest (upper
      // tiles, on the helper stream).  The next block's part-one update overlaps this block's part two in
      // memory, so it waits for it.
      const int c_lo = o0 > NBO ? o0 - NBO : 0;
      if (ob + 1 <= nob - 1) chk(hipStreamWaitEvent(s, side->events[2 * nob + ob + 1], 0));
      chk(launch_gemm_i8s(Vs, 0, Vs, c_lo, F + c_lo, ldf, o0, o0 - c_lo, wo, -1.0, 1, 0, s));
      // ---- inverse chain
      chk(hipStreamWaitEvent(sb, ev_factored, 0));
      chk(launch_gemm_i8s(Vs, 0, Vs, 0, F, ldf, c_lo, c_lo, wo, -1.0, 1, 1, sb));
      if (ob >= 1) chk(hipEventRecord(side->events[2 * nob + ob], sb));
      double* FJ = F + (int64_t)o0 * ldf + o1;                  // block row OB right of the diagonal block
      chk(launch_slice_i8(FJ, 1, ldf, ni - o1, wo, RJs, sb));   // R_OB,J (digits per column of it)
      chk(launch_slice_i8(Uob, NBO, 1, wo, wo, Urow, sb));
      chk(launch_gemm_i8s(Urow, 0, RJs, 0, FJ, ldf, wo, ni - o1, wo, 1.0, 0, 0, sb));           // U_OB,J = U_OB,OB R_OB,J
      chk(launch_slice_i8(FJ, 1, ldf, ni - o1, wo, RJs, sb));                                    // now U_OB,J
      chk(launch_gemm_i8s(Vs, 0, RJs, 0, F + o1, ldf, o0, ni - o1, wo, -1.0, 1, 0, sb));         // R_I,J -= V_I,OB U_OB,J
      chk(launch_gemm_i8s(Vs, 0, Ucol, 0, F + o0, ldf, o0, wo, wo, -1.0, 0, 0, sb));             // R_I,OB = -V_I,OB U_OB,OB
      chk(hipGetLastError());
      if (ob >= 2) chk(hipEventRecord(ev_inverted, sb));       // (the join is behind the last two)
    }
    // join: everything after the sweep runs on the caller's stream, and whatever the helper stream was given is behind it when
    // the call returns, also if a launch or an event call failed part-way
    hipEvent_t ev_join = side->events[3 * nob + 1];
    hipError_t joined = hipEventRecord(ev_join, sb);
    if (joined == hipSuccess) joined = hipStreamWaitEvent(s, ev_join, 0);
    chk(joined);
    if (!ok) return GPTAQ_ELAUNCH;
  }
  // U -> H (fp32) and the bf16 splits.
  hipLaunchKernelGGL(extract_U_kernel, dim3((unsigned)(np / 64), (unsigned)(np / 64)), dim3(256), 0, s, F, ldf, ni, H,
                     ldh, Uh, Ul, Uth, Utl, np);
  GPTAQ_LAUNCH_CHECK();
  // The K ranges of these two products are triangular, so tiles differ in length by the whole of K: the tile list is
  // dealt to the XCDs four tiles at a time (`deal`), not in contiguous runs (n = 11008: 2.8 -> 1.2 ms per product), and
  // while 256-tiles make a single round, the longest one sets the time and 128-tiles balance better (n = 4096)
  const int t256 = gemm_tile_for(n, n);
  const int tile = (t256 == 256 && (np / 256) * (np / 256) <= 256) ? 128 : t256;
  GemmBatch b{};
  b.nprob = 1; b.tile = tile;
  GemmProblem& g = b.p[0];
  // O = triu(dXXT U^T, 1): O[i][a] = sum_{b >= a} dXXT[i][b] U[a][b]
  g.C = Obuf; g.ldc = np; g.M = ni; g.N = ni; g.K = (int)np;
  g.tiles_m = g.tiles_n = (int)(np / tile);
  g.kind = 2; g.nterm = 1; g.tile_mode = 1; g.k_mode = 1; g.store_mode = 2; g.deal = 1;
  g.term[0] = {{Ah, Al}, {Uh, Ul}, 32, 32, np * 32, np * 32};
  hipError_t e;
  {
    ProfScope ps(kProfPGemm, s);
    e = launch_gemm(b, s);
  }
  if (e != hipSuccess) { set_last_hip_error(e); return GPTAQ_ELAUNCH; }
  // split O (reuses the dXXT split buffers), then P = O U: P[i][j] = sum_{i < a <= j} O[i][a] U[a][j]
  hipLaunchKernelGGL(split_rows_kernel, dim3((unsigned)((np + 255) / 256), (unsigned)(np / 4)), dim3(256), 0, s, Obuf, np,
                     ni, (const uint8_t*)nullptr, Ah, Al, np, (int32_t*)nullptr);
  GPTAQ_LAUNCH_CHECK();
  g.C = dXXT; g.ldc = ldh; g.k_mode = 2;
  g.term[0] = {{Ah, Al}, {Uth, Utl}, 32, 32, np * 32, np * 32};
  {
    ProfScope ps(kProfPGemm, s);
    e = launch_gemm(b, s);
  }
  if (e != hipSuccess) { set_last_hip_error(e); return GPTAQ_ELAUNCH; }
  return GPTAQ_OK;
}
