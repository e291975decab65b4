// The factor sweep of Algorithm 1, line 3 (see prepare.hip for the arithmetic): launches on one stream, each with a part of the
// sequential chain and, in further workgroups, products of the blocks before that the chain has no need of yet.
//
// An outer block OB of 256 columns is two launches (o0: its first column; t: OB, t + 1, t + 2: the blocks before it):
//
//   launch     chain                                              beside it
//   1 factor   F_OB,OB = V V^T in one workgroup, its second       t + 1: U_OB,J = U_OB,OB R_OB,J, R_I,OB = -V_I,OB U_OB,OB and
//     and      half's tile rows in eight more, and behind the     F_II -= V_I,OB V_I,OB^T but for the column block that S did; t + 2:
//     panel    products V_I,OB and U_OB,OB as digits              R_I,J -= V_I,OB U_OB,J, rows above OB(t + 1)
//   2 S        F_I,next -= V_I,OB V_next,OB^T                     digits of the rows of U_OB,OB; t + 1: R_I,J -= V_I,OB U_OB,J for the
//                                                                 rows of OB(t); what is left of t + 2 above OB(t)
//
// A launch waits for all of the one before, which costs about 1 us; nothing else orders the two kinds of work.  (With the products
// on a helper stream and events in between, a block of a small matrix took 102 us, of which 27 were events: a record costs
// the stream 3 us, a wait for another stream's event 9, however long ago that was reached.)
#include "common.h"
#include "factor_roles.h"
#include "gemm_i8s.h"
#include "factor_sweep.h"
#include <algorithm>

namespace gptaq {

namespace {
constexpr int kSweepProducts = 4;
struct SweepLaunch {
  BlockFactor f;
  BlockPanel p;
  I8RowBlock row_block;
  I8Slice slice;
  I8Gemm product[kSweepProducts];
  SplitRows split;
  // workgroups, in this order: chain, row block, slice, products (each from a multiple of 8 on: a workgroup's XCD is its number
  // modulo 8), split, and the chain's panel, which has to wait for the factorisation
  int32_t chain_end, row_block_end, slice_end, product_at[kSweepProducts], product_wgs[kSweepProducts], split_at, split_columns, panel_at;
};

constexpr int kSweepLds = std::max({(int)(Shape<64>::NSTAGE * Shape<64>::STAGE), (int)sizeof(FactorShared), (int)sizeof(PanelShared),
                                    (int)sizeof(RowBlockShared), (int)sizeof(SliceShared)});
static_assert(kSweepLds <= 80 * 1024, "two workgroups to a CU");

__global__ __launch_bounds__(256, 2) void sweep_kernel(SweepLaunch a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int wg = blockIdx.x;
  if (wg < a.chain_end || wg >= a.panel_at) {
    __shared__ int number;
    if (threadIdx.x == 0) number = atomicAdd(a.f.sync + BlockSync::kTicket, 1);
    __syncthreads();
    const int id = number;
    if (id == 0) factor_role(a.f, *reinterpret_cast<FactorShared*>(smem));
    else if (id < kFactorTeam) half_row_role(a.f, id - 1, *reinterpret_cast<PanelShared*>(smem));
    else panel_role(a.f, a.p, id - kFactorTeam, *reinterpret_cast<PanelShared*>(smem));
    return;
  }
  if (wg < a.row_block_end) {
    row_block_i8(a.row_block, wg - a.chain_end, *reinterpret_cast<RowBlockShared*>(smem));
    return;
  }
  if (wg < a.slice_end) {
    slice_i8(a.slice, wg - a.row_block_end, *reinterpret_cast<SliceShared*>(smem));
    return;
  }
  if (wg >= a.split_at) {
    const int id = wg - a.split_at;
    split_rows(a.split, id % a.split_columns, id / a.split_columns);
    return;
  }
  int q = kSweepProducts - 1;
  while (q > 0 && wg < a.product_at[q]) --q;
  const int id = wg - a.product_at[q];
  if (id >= 0 && id < a.product_wgs[q]) multiply_i8<64>(a.product[q], id, a.product_wgs[q], smem);
}

// products too large for 64-row tiles, in a launch of their own
__global__ __launch_bounds__(256, 1) void multiply_i8_kernel(I8Gemm g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  multiply_i8<128>(g, blockIdx.x, gridDim.x, smem);
}

// Workgroups per product and launch, at most (for BM = 128; twice as many of the half-size ones), each walking several tiles: very large
// products (n >= 28672) run tens of tiles per workgroup.
constexpr int kI8Workgroups = 1024;

// Which shape: measured with K = 256, 64-row tiles against 128-row tiles: 25.7 / 32.7 us for a 10752 x 256 update,
// 193 / 220 for 5376^2, 461 / 505 for the upper half of 10752^2, 3040 / 3038 for the upper half of 26624^2,
// 3245 / 3046 for 40960 x 8192.  The small tiles win while latencies matter and lose a little once the product is
// large enough to be bound by its traffic.
constexpr int64_t kI8SmallProduct = (int64_t)1 << 28;     // M * N up to here: 64-row tiles

// C = beta C + alpha A B^T over rows [a_row0, a_row0 + M) of A and [b_row0, b_row0 + N) of B (offsets multiples of 128 and 64);
// upper_only skips the tiles entirely below the diagonal of C.
struct Product {
  I8Gemm g{};                                    // tile0, ntile: what is left of the list
  int bm = 64;
  bool bad = false;
  int left() const { return g.ntile; }
  I8Gemm take(int tiles) {
    I8Gemm p = g;
    p.ntile = tiles < g.ntile ? tiles : g.ntile;
    g.tile0 += p.ntile;
    g.ntile -= p.ntile;
    return p;
  }
};
Product product(const I8Operand& A, int a_row0, const I8Operand& B, int b_row0, double* C, int64_t ldc, int M, int N, int K, double alpha,
                int beta, int upper_only) {
  Product r;
  if (M <= 0 || N <= 0 || K <= 0) return r;
  const bool small = (int64_t)M * N <= kI8SmallProduct;
  const int bm = small ? 64 : 128, ahead = small ? Shape<64>::AHEAD : Shape<128>::AHEAD;
  I8Gemm& g = r.g;
  r.bm = bm;
  g.tiles_m = (M + bm - 1) / bm;
  g.tiles_n = (N + BN - 1) / BN;
  r.bad = K > kI8MaxK || a_row0 % 128 || b_row0 % BN || a_row0 + g.tiles_m * bm > A.rows_pad || b_row0 + g.tiles_n * BN > B.rows_pad;
  g.A = A.planes + (int64_t)a_row0 * KC; g.a_plane = A.plane_stride(); g.a_chunk = A.chunk_stride(); g.sa = A.scale + a_row0;
  g.B = B.planes + (int64_t)b_row0 * KC; g.b_plane = B.plane_stride(); g.b_chunk = B.chunk_stride(); g.sb = B.scale + b_row0;
  g.C = C; g.ldc = ldc; g.M = M; g.N = N; g.beta = beta; g.upper_only = upper_only;
  const int nch = (K + KC - 1) / KC;             // (a sliced operand is zero past its K)
  g.nchunk = nch < ahead ? ahead : nch;
  g.alpha = alpha;
  for (int first = 0; first < g.tiles_m; first += 4) {
    const int gsz = g.tiles_m - first < 4 ? g.tiles_m - first : 4;
    const int c0 = upper_only ? (first * (bm / BN) < g.tiles_n ? first * (bm / BN) : g.tiles_n) : 0;
    g.ntile += gsz * (g.tiles_n - c0);
  }
  return r;
}

constexpr int kBesideS = 128;                    // tiles that fit beside S without holding it up

// One launch, put together part by part.
struct Step {
  SweepLaunch a{};
  int products = 0, slice_wgs = 0, row_block_wgs = 0, chain_wgs = 0, panel_wgs = 0, split_wgs = 0;
  bool bad = false;
  void row_block(const I8RowBlock& r) {
    if (r.J <= 0) return;
    bad |= r.wo > kI8MaxK || r.wo > r.Urow.rows_pad || round_up(r.J, 32) > r.out.rows_pad;
    a.row_block = r;
    row_block_wgs = (r.J + 31) / 32;
  }
  void slice(const double* src, int64_t sr, int64_t sk, int R, int K, const I8Operand& o) {
    if (R <= 0) return;
    bad |= K > kI8MaxK || (sr != 1 && sk != 1) || R > o.rows_pad;
    a.slice = I8Slice{src, sr, sk, R, K, o};
    slice_wgs = (R + 31) / 32;
  }
  // up to `tiles` of what is left of p; the number taken
  int multiply(Product& p, int tiles) {
    bad |= p.bad;
    if (tiles <= 0 || p.left() == 0) return 0;
    a.product[products] = p.take(tiles);
    const int n = a.product[products].ntile;
    a.product_wgs[products++] = n < 2 * kI8Workgroups ? n : 2 * kI8Workgroups;
    return n;
  }
  hipError_t launch(hipStream_t s) {
    static LdsLimitOnce lds;
    if (bad) return hipErrorInvalidValue;
    int at = a.chain_end = chain_wgs;
    at = a.row_block_end = at + row_block_wgs;
    at = a.slice_end = at + slice_wgs;
    for (int i = 0; i < kSweepProducts; ++i) {
      if (i < products) at = (at + 7) / 8 * 8;
      a.product_at[i] = at;
      at += a.product_wgs[i];
    }
    a.split_at = at;
    at = a.panel_at = at + split_wgs;
    at += panel_wgs;
    if (at == 0) return hipSuccess;
    const hipError_t e = lds.ensure((const void*)&sweep_kernel, kSweepLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sweep_kernel, dim3((unsigned)at), dim3(256), kSweepLds, s, a);
    return hipGetLastError();
  }
};

hipError_t launch_large(Product& p, hipStream_t s) {
  using S = Shape<128>;
  static LdsLimitOnce lds;
  if (p.bad) return hipErrorInvalidValue;
  const hipError_t e = lds.ensure((const void*)&multiply_i8_kernel, S::NSTAGE * S::STAGE);
  if (e != hipSuccess) return e;
  const I8Gemm g = p.take(p.left());
  hipLaunchKernelGGL(multiply_i8_kernel, dim3((unsigned)(g.ntile < kI8Workgroups ? g.ntile : kI8Workgroups)), dim3(256), S::NSTAGE * S::STAGE, s, g);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_factor_sweep(const FactorSweep& w, hipStream_t s) {
  const int n = w.n, nob = (n + kFactorBlock - 1) / kFactorBlock;
  hipError_t err = hipSuccess;
  auto go = [&](Step& st) { if (err == hipSuccess) err = st.launch(s); };
  auto large = [&](Product& p) { if (p.bm == 128 && p.left() && err == hipSuccess) err = launch_large(p, s); };
  // what is left to do of the block before, and of the one before that
  I8RowBlock row_block{};
  Product close, schur, near, far;
  for (int ob = nob - 1; ob >= 0; --ob) {
    const int o0 = ob * kFactorBlock, o1 = n < o0 + kFactorBlock ? n : o0 + kFactorBlock, wo = o1 - o0;
    const I8Operand& Vs = w.Vs[ob % 3];
    large(schur);
    large(far);
    const int p1 = n < o1 + kFactorBlock ? n : o1 + kFactorBlock;      // R_I,J -= V_I,OB U_OB,J of the block before, in rows of F
    auto update = [&](int row0, int rows) {
      return product(w.Vs[(ob + 1) % 3], row0, w.UJ[(ob + 1) & 1], 0, w.F + (int64_t)row0 * w.ldf + p1, w.ldf, rows, n - p1, p1 - o1, -1.0, 1, 0);
    };
    {
      Step st;
      st.a.f = BlockFactor{w.F, w.ldf, n, o0, w.info, w.V, w.T, w.sync + ob * (kBlockSyncBytes / 4)};
      st.a.p = BlockPanel{Vs, w.Ucol[ob & 1], w.Uob, w.F + (int64_t)o0 * w.ldf + o0};
      st.chain_wgs = kFactorTeam;
      st.panel_wgs = NT + o0 / 16;
      if (ob == nob - 1) {                       // dXXT's split depends on nothing here
        st.a.split = w.split;
        st.a.split_columns = (int)((w.split.np + 255) / 256);
        st.split_wgs = (int)(w.split.np / kSplitRowsPerWg) * st.a.split_columns;
      }
      st.row_block(row_block);
      st.multiply(near, near.left());
      st.multiply(close, close.left());
      st.multiply(schur, schur.left());
      st.multiply(far, far.left() - kBesideS);
      go(st);
    }
    const int c_lo = o0 > kFactorBlock ? o0 - kFactorBlock : 0;
    {
      Step st;
      Product next = product(Vs, 0, Vs, c_lo, w.F + c_lo, w.ldf, o0, o0 - c_lo, wo, -1.0, 1, 0), rest;
      if (ob < nob - 1) rest = update(o0, wo);
      if (o1 < n) st.slice(w.Uob, 1, kFactorBlock, wo, wo, w.Urow);
      st.multiply(next, next.left());
      st.multiply(rest, rest.left());
      st.multiply(far, far.left());
      go(st);
    }
    if (ob < nob - 1) {
      near = update(c_lo, o0 - c_lo);
      far = update(0, c_lo);
    }
    schur = product(Vs, 0, Vs, 0, w.F, w.ldf, c_lo, c_lo, wo, -1.0, 1, 1);
    close = product(Vs, 0, w.Ucol[ob & 1], 0, w.F + o0, w.ldf, o0, wo, wo, -1.0, 0, 0);                        // R_I,OB = -V_I,OB U_OB,OB
    row_block = I8RowBlock{w.F + (int64_t)o0 * w.ldf + o1, w.ldf, n - o1, wo, w.Urow, w.UJ[ob & 1]};
  }
  Step last;
  last.row_block(row_block);
  go(last);
  return err;
}

}  // namespace gptaq
