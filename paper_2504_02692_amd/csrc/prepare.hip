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
//     factor : F_OB,OB = V_OB,OB V_OB,OB^T                                    } fp64 (factor_roles.h)
//     panel  : V_I,OB = F_I,OB V_OB,OB^-T and U_OB,OB = V_OB,OB^-1, as digits }
//     syrk   : F_II  -= V_I,OB V_I,OB^T                (rank 256)  } the n^3 * 2/3 bulk: digit-sliced operands,
//     rowblk : U_OB,J  = U_OB,OB R_OB,J                            } exact int8 MFMA products,
//     rupd   : R_I,J  -= V_I,OB U_OB,J                 (rank 256)  } fp64 recombination (gemm_i8s.h)
//     close  : R_I,OB  = -V_I,OB U_OB,OB
//
// Theorem 4.2's two products then run on the bf16 MFMA GEMM with fp32 operands split into
// bf16 hi+lo (three cross products per term).
#include "common.h"
#include "factor_sweep.h"

namespace gptaq {

constexpr int NBO = kFactorBlock;             // outer block (columns per rank-256 update)

// ----------------------------------------------------------------------------- statistics
// One workgroup: dead inputs, lambda = damp * mean(diag), info words; the factor sweep's flags are cleared.
__global__ __launch_bounds__(1024) void diag_stats_kernel(const float* H, int64_t ldh, int n, float damp,
                                                          uint8_t* dead, double* lam_out, int32_t* info, int32_t* sync,
                                                          int nsync) {
  for (int i = threadIdx.x; i < nsync; i += 1024) sync[i] = 0;
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
// 256 columns of 16 rows, one workgroup: a wavefront four rows, four columns a lane.  Bound by memory: 30 us at n = 4096, 139 at
// 11008 (one entry a thread: 36 and 205).
constexpr int kBuildRows = 16;
__global__ __launch_bounds__(256) void build_F_kernel(const float* H, int64_t ldh, int n, const double* lam, double* F, int64_t ldf, int32_t* info) {
  typedef __attribute__((ext_vector_type(2))) double f64x2;
  const int j = blockIdx.x * 256 + 4 * (threadIdx.x & 63), r0 = kBuildRows * blockIdx.y + 4 * (threadIdx.x >> 6);
  if (blockIdx.x * 256 + 256 <= kBuildRows * blockIdx.y || j >= n) return;
  const bool wide = ((uintptr_t)H & 15) == 0 && ldh % 4 == 0 && j + 4 <= n;
  float h[4][4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float* src = H + (int64_t)min(r0 + q, n - 1) * ldh;
    if (wide) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(src + j);
#pragma unroll
      for (int e = 0; e < 4; ++e) h[q][e] = x[e];
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) h[q][e] = src[min(j + e, n - 1)];
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = r0 + q;
    if (i >= n || j + 3 < i) continue;
    double v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = (double)h[q][e];
      if (j + e >= i && j + e < n && !__builtin_isfinite(h[q][e])) atomicMin(info, -(1 + i));
      if (j + e == i) {
        if (v[e] == 0.0) v[e] = 1.0;
        v[e] += *lam;
      }
    }
    // (what lies below the diagonal or past column n in a row of F is not read, and F's rows are a multiple of 16 long)
    double* dst = F + (int64_t)i * ldf + j;
    *reinterpret_cast<f64x2*>(dst) = f64x2{v[0], v[1]};
    *reinterpret_cast<f64x2*>(dst + 2) = f64x2{v[2], v[3]};
  }
}

// --------------------------------------------------------------- extraction and splits
// U (fp32, upper, zeros below) from F; its bf16 hi/lo split row-major (Uh, Ul) and
// transposed (Uth, Utl), zero-padded to np x np.   grid (np/64, np/64).
// Bound by memory at large n, by the latency of its loads at small: with 256 threads, 16 rows each in turn, 9 / 41 / 297 us at
// n = 512 / 4096 / 11008; 5 / 38 / 257.
constexpr int kExtractThreads = 1024, kExtractStep = kExtractThreads / 64;
__global__ __launch_bounds__(kExtractThreads) void extract_U_kernel(const double* F, int64_t ldf, int n, float* U, int64_t ldu, uint16_t* Uh,
                                                                    uint16_t* Ul, uint16_t* Uth, uint16_t* Utl, int64_t np) {
  __shared__ uint16_t th[64][66], tl[64][66];
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  const int c = threadIdx.x & 63, rb = threadIdx.x >> 6, gc = c0 + c;
  if (c0 / kSplitBlock < r0 / kSplitBlock) {
#pragma unroll
    for (int p = 0; p < 64 / kExtractStep; ++p) {
      const int gr = r0 + rb + kExtractStep * p;
      if (gr < n && gc < n) U[(int64_t)gr * ldu + gc] = 0.f;
    }
    return;
  }
  double f[64 / kExtractStep];
#pragma unroll
  for (int p = 0; p < 64 / kExtractStep; ++p) f[p] = F[(int64_t)min(r0 + rb + kExtractStep * p, n - 1) * ldf + min(gc, n - 1)];
#pragma unroll
  for (int p = 0; p < 64 / kExtractStep; ++p) {
    const int r = rb + kExtractStep * p, gr = r0 + r;
    const float u = gr < n && gc < n && gc >= gr ? (float)f[p] : 0.f;
    if (gr < n && gc < n) U[(int64_t)gr * ldu + gc] = u;
    const uint16_t h = bf16_rne(u);
    const uint16_t l = bf16_rne(u - bf16_f32(h));
    const int64_t o = operand_at(gr, gc, np);
    Uh[o] = h;
    Ul[o] = l;
    th[r][c] = h;
    tl[r][c] = l;
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 64 / kExtractStep; ++p) {
    const int r = rb + kExtractStep * p;            // r: column of U inside the tile, c: row of U
    const int64_t o = operand_at(c0 + r, r0 + c, np);
    Uth[o] = th[c][r];
    Utl[o] = tl[c][r];
  }
}

}  // namespace gptaq

using namespace gptaq;

namespace {
struct PrepLayout {
  int64_t np;
  int64_t rp;                      // rows of a sliced operand that spans the whole matrix
  size_t off_F, off_lam, off_dead, off_O, off_b[6], off_Uob, off_V, off_T, off_sync, off_pl[8], off_sc[8], total;
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
  L.off_Uob = take((size_t)NBO * NBO * 8);
  L.off_V = take(kFactorTileBytes);
  L.off_T = take(kHalfTileBytes);
  L.off_sync = take((size_t)((n + NBO - 1) / NBO) * kBlockSyncBytes);
  // sliced operands of the rank-256 products: V_I,OB (three blocks' in turn), U_OB,J (two blocks'), and U_OB,OB by columns (two) and
  // by rows
  L.rp = round_up(n, 128);
  for (int i = 0; i < 8; ++i) {
    const int64_t rows = i < 5 ? L.rp : NBO;
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
  uint16_t *Oh = (uint16_t*)(base + L.off_O), *Ol = Oh + L.np * L.np;      // O as the left operand of the last product
  int32_t* sync = (int32_t*)(base + L.off_sync);
  I8Operand sl[8];
  for (int i = 0; i < 8; ++i) sl[i] = I8Operand{base + L.off_pl[i], (int32_t*)(base + L.off_sc[i]), i < 5 ? L.rp : (int64_t)NBO};
  const int64_t ldf = round_up(n, 16);
  uint16_t* bb[6];
  for (int i = 0; i < 6; ++i) bb[i] = (uint16_t*)(base + L.off_b[i]);
  const int64_t np = L.np;
  uint16_t *Uh = bb[0], *Ul = bb[1], *Uth = bb[2], *Utl = bb[3], *Ah = bb[4], *Al = bb[5];
  const int ni = (int)n;

  hipLaunchKernelGGL(diag_stats_kernel, dim3(1), dim3(1024), 0, s, H, ldh, ni, damp, deadbuf, lam, info, sync,
                     (int)((n + NBO - 1) / NBO * (kBlockSyncBytes / 4)));
  GPTAQ_LAUNCH_CHECK();
  hipLaunchKernelGGL(build_F_kernel, dim3((unsigned)((n + 255) / 256), (unsigned)((n + kBuildRows - 1) / kBuildRows)), dim3(256), 0, s, H, ldh, ni,
                     lam, F, ldf, info);
  GPTAQ_LAUNCH_CHECK();

  {
    ProfScope sweep_scope(kProfFactor, s);
    // (dXXT, dead rows zeroed, is split for the products at the end on the way)
    const hipError_t swept = launch_factor_sweep(
        FactorSweep{F, ldf, ni, info, (double*)(base + L.off_V), (double*)(base + L.off_T), (double*)(base + L.off_Uob), sync,
                    {sl[0], sl[1], sl[2]}, {sl[3], sl[4]}, {sl[5], sl[6]}, sl[7], SplitRows{dXXT, ldh, ni, deadbuf, Ah, Al, np, info}}, s);
    if (swept != hipSuccess) { set_last_hip_error(swept); return GPTAQ_ELAUNCH; }
  }
  // U -> H (fp32) and the bf16 splits.
  hipLaunchKernelGGL(extract_U_kernel, dim3((unsigned)(np / 64), (unsigned)(np / 64)), dim3(kExtractThreads), 0, s, F, ldf, ni, H,
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
  g.C = nullptr; g.ldc = np; g.M = ni; g.N = ni; g.K = (int)np;
  g.tiles_m = g.tiles_n = (int)(np / tile);
  g.kind = 2; g.nterm = 1; g.tile_mode = 1; g.k_mode = 1; g.store_mode = 3; g.out_hi = Oh; g.out_lo = Ol; g.deal = 1;
  g.term[0] = {{Ah, Al}, {Uh, Ul}, 32, 32, np * 32, np * 32};
  hipError_t e;
  {
    ProfScope ps(kProfPGemm, s);
    e = launch_gemm(b, s);
  }
  if (e != hipSuccess) { set_last_hip_error(e); return GPTAQ_ELAUNCH; }
  // P = O U: P[i][j] = sum_{i < a <= j} O[i][a] U[a][j]
  g.C = dXXT; g.ldc = ldh; g.k_mode = 2; g.store_mode = 2;
  g.term[0] = {{Oh, Ol}, {Uth, Utl}, 32, 32, np * 32, np * 32};
  {
    ProfScope ps(kProfPGemm, s);
    e = launch_gemm(b, s);
  }
  if (e != hipSuccess) { set_last_hip_error(e); return GPTAQ_ELAUNCH; }
  return GPTAQ_OK;
}
