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

__global__ __launch_bounds__(256) void split_rows_kernel(SplitRows a) { split_rows(a, blockIdx.x, blockIdx.y); }

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
  float* Obuf = (float*)(base + L.off_O);
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
  hipLaunchKernelGGL(build_F_kernel, dim3((unsigned)((n + 255) / 256), (unsigned)n), dim3(256), 0, s, H, ldh, ni,
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
  hipLaunchKernelGGL(split_rows_kernel, dim3((unsigned)((np + 255) / 256), (unsigned)(np / kSplitRowsPerWg)), dim3(256), 0, s,
                     SplitRows{Obuf, np, ni, nullptr, Ah, Al, np, nullptr});
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
