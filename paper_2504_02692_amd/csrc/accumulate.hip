// Algorithm 1, line 2:  H += X X^T,  dXXT += (X~ - X) X^T, streamed over token chunks.
//
// Two steps per chunk.  (1) A bandwidth-bound pass reads the token-major bf16 X and X~,
// forms dX = X~ - X in fp32, splits it exactly into two bf16 terms (hi = rne(dX),
// lo = dX - hi) and writes X, hi, lo transposed in k-tile-major order: [token tile of 32]
// [neuron][32 tokens], the operand layout the MFMA GEMM wants (tokens are its K dimension and
// a block of neurons x one token tile is a single contiguous run).  From 1921 columns on lo is written as a sparse operand
// (sparse_remainder, GemmTerm).
// (2) One launch of the MFMA GEMM computes dXXT += hi X^T + lo X^T on all tiles and
// H += X X^T on the tiles that touch the upper triangle.
#include "common.h"
#include <mutex>

namespace gptaq {

// Workspace of gptaq_accumulate_noalloc: one copy per GPU, owned by the code object, never freed.
constexpr size_t kScratchBytes = (size_t)32 << 20;
constexpr int64_t kScratchMaxN = 16384;                   // 6 * 16384 * 320 tokens still fit
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

__device__ __forceinline__ float bf16_to_f32(uint32_t h) { return __uint_as_float(h << 16); }
__device__ __forceinline__ uint32_t f32_to_bf16_rne(float f) {
  __bf16 b = (__bf16)f;                       // v_cvt_pk_bf16_f32: round to nearest even
  return (uint32_t)__builtin_bit_cast(uint16_t, b);
}

// grid: (n_pad / 64, c_pad / 64).  Writes zeros where the source is out of range, so the
// GEMM can run on whole tiles.
// SPARSE: lo in the form of GemmTerm's kind 3 (sparse_remainder), else like hi.
template <bool SPARSE>
__global__ __launch_bounds__(256) void split_transpose_kernel(
    const uint16_t* __restrict__ X, const uint16_t* __restrict__ Xt, int64_t ldx,
    int tokens, int n, uint16_t* __restrict__ oX, uint16_t* __restrict__ oHi,
    uint16_t* __restrict__ oLo, uint16_t* __restrict__ oLo2, int64_t ldo /* padded rows */, int tile0 /* first 64-token tile of the output */,
    const int32_t* __restrict__ row_of /* NULL, or operand row of input column j (a permutation of 0 .. n-1) */) {
  constexpr int LS = 72;                                  // padded LDS row, 144 bytes
  __shared__ __attribute__((aligned(16))) uint16_t sx[64 * LS], sh[64 * LS], sl[64 * LS];
  const int n0 = blockIdx.x * 64, t0 = blockIdx.y * 64;
  const int tid = threadIdx.x, r = tid >> 3, c = tid & 7;
  auto row_to = [&](int i) {                                // the operand row of input column n0 + i
    int64_t row = n0 + i;                                   // (padding rows stay where they are)
    if (row_of && row < n) {
      const int32_t rr = row_of[row];
      if (rr >= 0 && rr < n) row = rr;                      // (an entry out of range cannot send a write out of bounds)
    }
    return row;
  };
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int t = t0 + r + 32 * p, col = n0 + c * 8;
    u32x4 a = {0, 0, 0, 0}, b = {0, 0, 0, 0};
    if (t < tokens && col < n) {
      a = *reinterpret_cast<const u32x4*>(X + (int64_t)t * ldx + col);
      b = *reinterpret_cast<const u32x4*>(Xt + (int64_t)t * ldx + col);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t xa = (a[e >> 1] >> ((e & 1) * 16)) & 0xffffu;
      const uint32_t xb = (b[e >> 1] >> ((e & 1) * 16)) & 0xffffu;
      const float d = bf16_to_f32(xb) - bf16_to_f32(xa);
      const uint32_t hi = f32_to_bf16_rne(d);
      const uint32_t lo = f32_to_bf16_rne(d - bf16_to_f32(hi));
      const int o = (c * 8 + e) * LS + r + 32 * p;
      sx[o] = (uint16_t)xa;
      sh[o] = (uint16_t)hi;
      sl[o] = (uint16_t)lo;
    }
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int nl = r + 32 * p;
    const int64_t g = (((int64_t)(blockIdx.y + tile0) * 2 + (c >> 2)) * ldo + row_to(nl)) * 32 + (c & 3) * 8;   // k-tile-major
    *reinterpret_cast<u32x4*>(oX + g) = *reinterpret_cast<const u32x4*>(sx + nl * LS + c * 8);
    *reinterpret_cast<u32x4*>(oHi + g) = *reinterpret_cast<const u32x4*>(sh + nl * LS + c * 8);
    if (!SPARSE) *reinterpret_cast<u32x4*>(oLo + g) = *reinterpret_cast<const u32x4*>(sl + nl * LS + c * 8);
  }
  if (!SPARSE) return;
  // lo, in the form that GemmTerm describes: a wavefront has a 32 x 32 block and a lane the 16 tokens of its row that it has there
  const int lane = tid & 63, nl = (tid >> 7) * 32 + (lane & 31), k = tid >> 6 & 1, half = lane >> 5;
  uint64_t q[4];
  int nz[4];
  bool more = false;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const u32x4 x = *reinterpret_cast<const u32x4*>(sl + nl * LS + k * 32 + half * 16 + h * 8);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const uint32_t a = x[2 * e], b = x[2 * e + 1];
      const int z = (a & 0x7fffu ? 1 : 0) | (a & 0x7fff0000u ? 2 : 0) | (b & 0x7fffu ? 4 : 0) | (b & 0x7fff0000u ? 8 : 0);
      q[2 * h + e] = (uint64_t)b << 32 | a;
      nz[2 * h + e] = z;
      more |= __builtin_popcount(z) > 2;
    }
  }
  const bool dense = __ballot(more) != 0;
  uint32_t v[4], v2[4], places = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    // places of two values that hold what is not zero: (0,1) (0,3) (1,3) (0,1) | (2,3) (0,2) (1,2) - | (2,3) (0,3) (1,3) - | (2,3) - - -
    const uint32_t at = dense ? 4u : (uint32_t)(0x444E4DCE498E4DC4ull >> (4 * nz[e]) & 15);
    v[e] = (uint32_t)(q[e] >> (16 * (at & 3)) & 0xffff) | (uint32_t)(q[e] >> (16 * (at >> 2))) << 16;
    v2[e] = dense ? (uint32_t)(q[e] >> 32) : e == 0 ? kRowMark : 0u;
    places |= at << (4 * e);
  }
  const int64_t kt = (int64_t)(blockIdx.y + tile0) * 2 + k;
  if (!row_of) {
    const int64_t row = n0 + nl;
    *reinterpret_cast<u32x4*>(oLo + (kt * ldo + row) * 16 + half * 8) = u32x4{v[0], v[1], v[2], v[3]};
    const int blk = (int)(row & 127) >> 5, piece = 2 * (lane & 31) + half;
    unsigned char* group = reinterpret_cast<unsigned char*>(oLo2 + (kt * ldo + (row & ~127)) * 16);
    places |= __shfl_down(places, 32) << 16;
    if (dense) {
      unsigned char* dst = piece == 0 ? group + 16 * blk : piece < 9 ? group + 64 + 128 * blk + 16 * (piece - 1) : group + 576 + 880 * blk + 16 * (piece - 9);
      *reinterpret_cast<u32x4*>(dst) = u32x4{v2[0], v2[1], v2[2], v2[3]};
    } else {
      if (half == 0) *reinterpret_cast<uint32_t*>(group + 64 + 128 * blk + 4 * lane) = places;
      if (lane == 0) *reinterpret_cast<uint32_t*>(group + 16 * blk) = kSparseMark;
    }
    return;
  }
  // by rows, in runs of 64 bytes as of hi and X  (a wavefront's rows are read and written by it alone)
  if (!dense) v2[0] |= places;
  *reinterpret_cast<u32x4*>(sl + nl * LS + k * 32 + half * 8) = u32x4{v[0], v[1], v[2], v[3]};
  *reinterpret_cast<u32x4*>(sl + nl * LS + k * 32 + 16 + half * 8) = u32x4{v2[0], v2[1], v2[2], v2[3]};
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int w = (tid >> 7) * 32 + (lane >> 2) + 16 * p;
    *reinterpret_cast<u32x4*>(oLo + (kt * ldo + row_to(w)) * 32 + (lane & 3) * 8) = *reinterpret_cast<const u32x4*>(sl + w * LS + k * 32 + (lane & 3) * 8);
  }
}

__global__ void symmetrize_kernel(float* H, int n, int64_t ldh) {
  __shared__ float t[32][33];
  const int bi = blockIdx.y, bj = blockIdx.x;
  if (bj < bi) return;                                     // handle pairs once, from the upper side
  const int i = bi * 32 + threadIdx.y, j = bj * 32 + threadIdx.x;
  if (i < n && j < n) t[threadIdx.y][threadIdx.x] = H[(int64_t)i * ldh + j];
  __syncthreads();
  const int li = bj * 32 + threadIdx.y, lj = bi * 32 + threadIdx.x;   // transposed position
  if (li < n && lj < n && li > lj) H[(int64_t)li * ldh + lj] = t[threadIdx.x][threadIdx.y];
}

// diag[j] += sum_t X[t][j]^2 (the diagonal of H) for the 32 columns of a workgroup: thread = (token lane, 8 columns),
// 64 token lanes; products of bf16 numbers are exact in fp32, the sums are taken in a fixed order.
__global__ __launch_bounds__(256) void column_sumsq_kernel(const uint16_t* __restrict__ X, int64_t ldx, int tokens, int n,
                                                           float* __restrict__ diag) {
  __shared__ float part[64][33];
  const int oct = threadIdx.x & 3, tl = threadIdx.x >> 2, col = blockIdx.x * 32 + oct * 8;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (col < n)
    for (int t = tl; t < tokens; t += 64) {
      const u32x4 a = *reinterpret_cast<const u32x4*>(X + (int64_t)t * ldx + col);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = bf16_to_f32((a[e >> 1] >> ((e & 1) * 16)) & 0xffffu);
        acc[e] = fmaf(x, x, acc[e]);
      }
    }
#pragma unroll
  for (int e = 0; e < 8; ++e) part[tl][oct * 8 + e] = acc[e];
  __syncthreads();
  if (threadIdx.x < 32 && blockIdx.x * 32 + threadIdx.x < n) {
    float sum = 0.f;
    for (int l = 0; l < 64; ++l) sum += part[l][threadIdx.x];
    diag[blockIdx.x * 32 + threadIdx.x] += sum;
  }
}

__global__ void invert_permutation_kernel(const int32_t* perm, int n, int32_t* inv) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r < n) {
    const int32_t i = perm[r];
    if (i >= 0 && i < n) inv[i] = r;
  }
}

// Whether the remainder's products are taken as sparse ones (kind 3): from 1921 columns on, where the upper form has more tiles than the
// chip has CUs.  dX does not fit a bf16 only where it is larger than the smaller of X and X~, so most of lo is zero: of its 32 x 32
// blocks 2 % are dense where X and X~ differ by 5 % of a channel's deviation, 14 % at 10 %, 38 % at 15, 69 % at 20, 96 % at 30, all at 50.  Fewer matrix
// instructions and operand bytes (41 KB instead of 48 for 32 tokens of a 256-tile, which is what bounds these launches).  By n alone: a staged
// call writes its operands before the number of tokens is known, and the sums do not depend on the form of the call.  Measured, us
// per call, dense operands / so, at differences of 5, 10, 20 and 50 %: 2048 columns and 32768 tokens 592 / 571, 597, 609, 627; 2736
// full 1275 / 1108, 1138, 1317, 1332; 3072 and 16384 594 / 487, 495, 547, 549; 4096 and 2048 138 / 105, 108, 117, 120; 4096 and 32768 1605 / 1383, 1431,
// 1576, 1640; 6144 and 16384 1600 / 1455, 1479, 1579, 1646; 11008 and 32768 9710 / 8803, 9032, 9699, 10081.  So where X~ is off by more than 20 % (with
// 128-tiles by more than 10) this is up to 5 % slower than dense operands: the sparse instruction draws more power, and positions are 2 % more bytes.  With fewer columns a
// workgroup has its CU to itself and the loop's branches show: 512 and 4096 tokens 54 / 58, 1536 and 4096 58 / 66.  Error of dXXT against 64
// bits 2.91e-7 (dense operands 2.96e-7) at 4104 columns and 6144 tokens.
static bool sparse_remainder(int64_t n) { const int64_t t = (n + 127) / 128; return t * (t + 1) > 256; }

// How many of H's last 256-tiles are taken as quarters: those past one tile for each of the 256 CUs, if they are few.  A tile of dXXT
// takes 1.45 times as long as one of H, so most CUs are idle while a second tile of H runs on a few of them.  A quarter fetches twice
// the bytes of its part of a tile: with many the launch takes longer (50 at 4352 columns: 1588 us to 1660).  Of the launches of 256-tiles only the upper
// form of 16 tile rows has few, 272 tiles (3841 to 4096 columns): 15 rows have 240, 17 306, and the full form 345 and more.  Measured, whole
// tiles / so, us: 4096 columns and 64 tokens 38 / 32, 512 53 / 45, 2048 118 / 101, 32768 1512 / 1390, 3848 and 32768 1485 / 1338.
static int quartered_tiles(int64_t tiles) {
  const int64_t more = tiles - 256;
  return more > 0 && more <= 32 ? (int)more : 0;
}

static int64_t padded_n(int64_t n) { return round_up(n, gemm_tile_for(n, n)); }

// The operands of `tokens` tokens (a multiple of 64) in a workspace: X, hi and lo of 2 bytes an entry, lo in the sparse form in two halves.
struct Operands {
  uint16_t *X, *hi, *lo, *lo2;
  size_t bytes;
  bool rows;               // lo by rows
};
static Operands operands_at(void* ws, int64_t np, int64_t tokens, bool rows) {
  const int64_t all = np * tokens;
  uint16_t* X = (uint16_t*)ws;
  return {X, X + all, X + 2 * all, X + 2 * all + all / 2, (size_t)(6 * all), rows};
}

// Whether the sums of a pass are taken in blocks of 32 x 64, a workgroup's wavefronts an eighth of the tokens each (launch_narrow_sums): up to
// 4096 tokens, where the full form has no more blocks than the chip has CUs (576 columns).  Measured, 128-tiles in one part or in parts
// (with a workspace for them) / so, us per call: n = 512 and 1024 tokens 21 / 16, 2048 25 / 21, 4096 53 or 32 / 32 (full form 53 or 32 / 29); 256 and 1024
// 19 / 15, 4096 50 or 27 / 28; with more tokens parts are the better (512 and 8192 40 / 47), and with a second block to a CU (640 and
// 4096, full form 33 / 45).  (By the full form alone: the upper form is bit for bit the full one where it is defined.)
static bool few_blocks(int64_t n, int64_t tokens) {
  const int64_t rows = (n + 31) / 32, cols = (n + 63) / 64;
  return tokens <= 4096 && rows * cols + cols * (cols + 1) <= 256;
}

// In how many parts of their tokens the sums of a pass are taken, and what the parts' sums need beside the operands.
// With few columns the tiles of H and dXXT leave most of the chip idle (n = 1024: 72 or 100 of 512 places for 128-tiles).  dXXT's tiles,
// of two products, are split in so many parts and H's, of one, in half as many, so that all workgroups take the same time.  (Four
// workgroups a tile row sum H's diagonal in one part: see diagonal_block.)  How many parts pay depends on how full the last round of 512
// workgroups is, which goes up and down with the tile rows: a line for each number of them.  Both forms of the call take the same
// number (the upper form is bit for bit the full one where it is defined), and there are more only with more tokens, so that the workspace of
// a call has room for every shorter one.  Measured, one part / so many, us per call, upper form (full):
//   columns  tokens
//    256      6144  72 / 33 (72 / 33)     32768  301 / 77 (314 / 77);  more parts than 8: the same
//    640      1536  28 / 26 (28 / 27)      2048  35 / 28 (35 / 28)     8192  93 / 42 (93 / 43)     32768  326 / 105 (331 / 110)
//    768      2048  36 / 29 (36 / 29)      8192  92 / 44 (92 / 55)    16384  172 / 76 (169 / 80)   32768  335 / 133 (326 / 153)
//    896      2048  36 / 30 (35 / 32)      6144  76 / 45 (76 / 50)    16384  178 / 87 (179 / 98)   32768  347 / 159 (349 / 180)
//   1024      1536  31 / 29 (30 / 31)      2048  35 / 29 (34 / 33)     8192  95 / 56 (94 / 75)     32768  384 / 196 (384 / 238)
//   1152      2048  37 / 34 (36 / 36)      6144  77 / 60 (78 / 65)    16384  184 / 106 (185 / 140) 32768  442 / 239 (436 / 302)
//   1280      4096  57 / 48 (57 / 54)     8192  100 / 80 (102 / 96)  16384  186 / 140 (186 / 172) 32768  487 / 261 (488 / 353)
//   1408      6144  80 / 66 (83 / 96)     16384  190 / 148 (196 / 202) 20480  240 / 174 (248 / 240)   32768  523 / 327 (519 / 388)
//   1536     16384  196 / 166 (214 / 230) 28672  468 / 309 (469 / 391) 32768  537 / 341 (536 / 444)
//   1664      6144  83 / 96 (116 / 105)   12288  153 / 150 (217 / 207) 23040  348 / 292 (379 / 373) 32768  546 / 410 (557 / 530)
//   1920     24576  432 / 361 (464 / 506) 32768  566 / 467 (626 / 661)
// One part stays where the best number makes one of the forms slower or gives little (in this list 1408 columns and 6144 or 16384 tokens, 1536 and
// 16384, 1664 and 6144 or 12288, 1920); at 1792 columns two would pay from 24576 tokens on (410 / 344 and 439 /
// 418).  Between two numbers of parts, where one form gains what the other loses (768 columns and 12288 tokens, 6 / 8 parts: 55 / 62 (73 / 64)),
// the line is where the sum of both does not care; at 1280 columns and 7488 tokens or more 2 parts serve the full form and 4 the upper one, which is the
// one in every solve whose columns keep their order: 8192 tokens, inputs from memory, 2 / 4 parts 94 / 90 (103 / 107), 16384 160 / 153 (173 / 182).  Errors
// against 64 bits fall with the length of the sums: dXXT 8.7e-7 to 2.4e-7 at n = 1024.
static int split_for(int64_t n, int64_t tokens) {
  if (sparse_remainder(n)) return 1;             // (remainder_loop takes all of K)
  if (few_blocks(n, tokens)) return 1;
  const int64_t t = (n + 127) / 128;
  if (t <= 3) return 8;                          // (more than 4096 tokens)
  static constexpr struct { int tokens, parts; } lines[][4] = {
      {{4160, 6}, {4736, 8}},                                    // 4 tile rows, up to 512 columns
      {{1728, 4}, {3072, 6}},                                    // 640
      {{1792, 4}, {8192, 6}, {14080, 8}, {27008, 12}},           // 768
      {{2048, 4}, {6912, 6}},                                    // 896
      {{2048, 4}, {16448, 8}},                                   // 1024
      {{2048, 2}, {4096, 4}, {14400, 6}},                        // 1152
      {{3072, 2}, {7488, 4}, {16768, 8}},                        // 1280
      {{18112, 4}, {23296, 6}},                                  // 1408
      {{28672, 8}},                                              // 1536
      {{23040, 6}},                                              // 1664
  };
  int parts = 1;
  if (t - 4 < (int64_t)(sizeof(lines) / sizeof(lines[0])))
    for (const auto& line : lines[t - 4])
      if (line.parts && tokens >= line.tokens) parts = line.parts;
  return parts;
}
static size_t partial_bytes(int64_t n, int split) {
  if (split <= 1) return 0;
  const int64_t t = (n + 127) / 128;
  return (size_t)(t * t * split + t * (t + 1) / 2 * (split / 2)) * (128 * 128 * 4);
}

}  // namespace gptaq

using namespace gptaq;

extern "C" size_t gptaq_accumulate_workspace_bytes(int64_t tokens, int64_t n) {
  if (tokens <= 0 || n <= 0) return 0;
  const int64_t c = round_up(tokens < 32768 ? tokens : 32768, 64);
  return (size_t)(3 * padded_n(n) * c * 2) + partial_bytes(n, split_for(n, c));
}

// The operands of c tokens, from 64-token tile `tile0` of o on.
static int launch_split(const Operands& o, const uint16_t* X, const uint16_t* Xtilde, int64_t ldx, int64_t c, int64_t n, int64_t np, int64_t tile0,
                        const int32_t* row_of, hipStream_t s) {
  ProfScope ps(kProfAccumSplit, s);
  hipLaunchKernelGGL(sparse_remainder(n) ? split_transpose_kernel<true> : split_transpose_kernel<false>,
                     dim3((unsigned)(np / 64), (unsigned)((c + 63) / 64)), dim3(256), 0, s, X, Xtilde, ldx, (int)c, (int)n, o.X, o.hi, o.lo, o.lo2,
                     np, (int)tile0, row_of);
  GPTAQ_LAUNCH_CHECK();
  return GPTAQ_OK;
}

// H += X X^T (upper tiles) and dXXT += (hi + lo) X^T over cp tokens of split operands, as one launch.
// dxxt_upper: only the tiles of dXXT that touch its upper triangle.  Eq. 17 masks dXXT L to its strictly upper part and
// L is lower triangular, so entry (i, k) of dXXT reaches P only through sums over k >= j > i: in the natural column
// order nothing on or below the diagonal is ever read, and two fifths of the products of the launch can be left out.
static hipError_t launch_products(const Operands& o, int64_t np, int64_t cp, int64_t n, float* H, float* dXXT, int64_t ldh, bool dxxt_upper,
                                  void* ws, size_t ws_bytes, hipStream_t s) {
  const int tile = gemm_tile_for(n, n);
  GemmBatch b{};
  b.nprob = 2;
  b.tile = tile;
  GemmProblem& a = b.p[0];
  a.C = dXXT; a.ldc = ldh; a.M = (int)n; a.N = (int)n; a.K = (int)cp;
  a.tiles_m = a.tiles_n = (int)(np / tile);
  a.kind = sparse_remainder(n) ? 3 : 1; a.nterm = 1; a.tile_mode = dxxt_upper ? 2 : 0; a.k_mode = 0; a.store_mode = 0;
  a.term[0] = {{o.hi, o.lo}, {o.X, o.lo2}, 32, 32, np * 32, np * 32};
  a.lo_rows = o.rows;
  GemmProblem& h = b.p[1];
  h = a;
  h.C = H; h.kind = 0; h.tile_mode = 2;
  h.term[0] = {{o.X, o.X}, {o.X, o.X}, 32, 32, np * 32, np * 32};
  if (a.kind == 3 && tile == 256) {
    const int64_t t = a.tiles_m, upper = t * (t + 1) / 2;
    h.quartered = quartered_tiles((dxxt_upper ? upper : t * t) + upper);
  }
  ProfScope ps(kProfAccumGemm, s);
  if (few_blocks(n, cp)) return launch_narrow_sums(b, s);
  const int split = split_for(n, cp);
  if (split > 1 && o.bytes + partial_bytes(n, split) <= ws_bytes) {      // (a smaller workspace: sums in one part)
    a.split = split;
    a.partial = (float*)((unsigned char*)ws + o.bytes);
    h.split = split / 2;
    h.partial = a.partial + (int64_t)a.tiles_m * a.tiles_m * split * (128 * 128);
  }
  return launch_gemm(b, s);
}

// the argument checks that need no workspace
static int accumulate_args(const uint16_t* X, const uint16_t* Xtilde, int64_t tokens, int64_t n, int64_t ldx, float* H,
                           float* dXXT, int64_t ldh) {
  if (!X || !Xtilde || !H || !dXXT) return GPTAQ_ENULL;
  if (tokens < 0 || n <= 0 || n % 8 || ldx < n || ldx % 8 || ldh < n || n > (1 << 20) ||
      tokens > (int64_t)1 << 30)
    return GPTAQ_EDIM;
  if (((uintptr_t)X | (uintptr_t)Xtilde) & 15) return GPTAQ_EDIM;
  return GPTAQ_OK;
}

static int accumulate_impl(const uint16_t* X, const uint16_t* Xtilde, int64_t tokens, int64_t n, int64_t ldx, float* H,
                           float* dXXT, int64_t ldh, bool dxxt_upper, void* ws, size_t ws_bytes, void* stream,
                           const int32_t* row_of = nullptr) {
  if (!ws) return GPTAQ_ENULL;
  if (const int rc = accumulate_args(X, Xtilde, tokens, n, ldx, H, dXXT, ldh)) return rc;
  if ((uintptr_t)ws & 255) return GPTAQ_EWORKSPACE;
  if (tokens == 0) return GPTAQ_OK;
  hipStream_t s = (hipStream_t)stream;
  const int64_t np = padded_n(n);
  int64_t cmax = (int64_t)(ws_bytes / (size_t)(6 * np)) / 64 * 64;
  if (cmax < 64) return GPTAQ_EWORKSPACE;
  if (cmax > 32768) cmax = 32768;    // keeps one fp32 running sum short (accuracy), and K in int32
  for (int64_t t0 = 0; t0 < tokens; t0 += cmax) {
    const int64_t c = tokens - t0 < cmax ? tokens - t0 : cmax;
    const int64_t cp = round_up(c, 64);
    const Operands o = operands_at(ws, np, cp, row_of != nullptr);
    if (const int rc = launch_split(o, X + t0 * ldx, Xtilde + t0 * ldx, ldx, c, n, np, 0, row_of, s)) return rc;
    hipError_t e = launch_products(o, np, cp, n, H, dXXT, ldh, dxxt_upper, ws, ws_bytes, s);
    if (e != hipSuccess) { set_last_hip_error(e); return GPTAQ_ELAUNCH; }
  }
  return GPTAQ_OK;
}

extern "C" int gptaq_accumulate(const uint16_t* X, const uint16_t* Xtilde, int64_t tokens,
                                int64_t n, int64_t ldx, float* H, float* dXXT, int64_t ldh,
                                void* ws, size_t ws_bytes, void* stream) {
  return accumulate_impl(X, Xtilde, tokens, n, ldx, H, dXXT, ldh, false, ws, ws_bytes, stream);
}

extern "C" int gptaq_accumulate_upper_permuted(const uint16_t* X, const uint16_t* Xtilde, int64_t tokens, int64_t n,
                                               int64_t ldx, const int32_t* inv_perm, float* H, float* dXXT, int64_t ldh,
                                               void* ws, size_t ws_bytes, void* stream) {
  if (!inv_perm) return GPTAQ_ENULL;
  return accumulate_impl(X, Xtilde, tokens, n, ldx, H, dXXT, ldh, true, ws, ws_bytes, stream, inv_perm);
}

extern "C" int gptaq_accumulate_diag(const uint16_t* X, int64_t tokens, int64_t n, int64_t ldx, float* diag, void* stream) {
  if (!X || !diag) return GPTAQ_ENULL;
  if (tokens < 0 || n <= 0 || n % 8 || ldx < n || ldx % 8 || n > (1 << 20) || tokens > (int64_t)1 << 30) return GPTAQ_EDIM;
  if ((uintptr_t)X & 15) return GPTAQ_EDIM;
  if (tokens == 0) return GPTAQ_OK;
  hipLaunchKernelGGL(column_sumsq_kernel, dim3((unsigned)((n + 31) / 32)), dim3(256), 0, (hipStream_t)stream, X, ldx,
                     (int)tokens, (int)n, diag);
  GPTAQ_LAUNCH_CHECK();
  return GPTAQ_OK;
}

extern "C" int gptaq_invert_permutation(const int32_t* perm, int64_t n, int32_t* inv, void* stream) {
  if (!perm || !inv) return GPTAQ_ENULL;
  if (n <= 0 || n > (1 << 24)) return GPTAQ_EDIM;
  hipLaunchKernelGGL(invert_permutation_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, perm,
                     (int)n, inv);
  GPTAQ_LAUNCH_CHECK();
  return GPTAQ_OK;
}

extern "C" int gptaq_accumulate_upper(const uint16_t* X, const uint16_t* Xtilde, int64_t tokens,
                                      int64_t n, int64_t ldx, float* H, float* dXXT, int64_t ldh,
                                      void* ws, size_t ws_bytes, void* stream) {
  return accumulate_impl(X, Xtilde, tokens, n, ldx, H, dXXT, ldh, true, ws, ws_bytes, stream);
}

// Device address of this GPU's copy of `scratch`, looked up once per device (with that device current).
// In host code the array's name is only a handle for this lookup, never an address to hand to a kernel.
static void* scratch_of_current_device() {
  static std::mutex mu;
  static void* ptr[64] = {nullptr};
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) { set_last_hip_error(e); return nullptr; }
    ptr[dev] = p;
  }
  return ptr[dev];
}

extern "C" int gptaq_accumulate_noalloc(const uint16_t* X, const uint16_t* Xtilde, int64_t tokens, int64_t n,
                                        int64_t ldx, float* H, float* dXXT, int64_t ldh, void* stream) {
  if (const int rc = accumulate_args(X, Xtilde, tokens, n, ldx, H, dXXT, ldh)) return rc;
  if (n > kScratchMaxN) return GPTAQ_ETOOLARGE;
  if (tokens == 0) return GPTAQ_OK;
  void* ws = scratch_of_current_device();
  if (!ws) return GPTAQ_ELAUNCH;
  // every pass overwrites the part of the scratch it reads (zero padding included), so nothing of the last
  // call's contents is ever read and nothing has to be cleared
  return accumulate_impl(X, Xtilde, tokens, n, ldx, H, dXXT, ldh, false, ws, kScratchBytes, stream);
}

static int accumulate_staged_impl(const uint16_t* X, const uint16_t* Xtilde, int64_t tokens, int64_t n, int64_t ldx,
                                  float* H, float* dXXT, int64_t ldh, bool dxxt_upper, void* ws, size_t ws_bytes,
                                  int64_t* pending, int flush, void* stream) {
  constexpr int64_t CAP = 32768;                 // tokens per product launch
  if (!H || !dXXT || !ws || !pending || (tokens > 0 && (!X || !Xtilde))) return GPTAQ_ENULL;
  if (tokens < 0 || n <= 0 || n % 8 || ldx < n || ldx % 8 || ldh < n || n > (1 << 20) || tokens > (int64_t)1 << 30 ||
      *pending < 0 || *pending >= CAP || *pending % 64 || (!flush && tokens % 64))
    return GPTAQ_EDIM;
  if (tokens > 0 && (((uintptr_t)X | (uintptr_t)Xtilde) & 15)) return GPTAQ_EDIM;
  const int64_t np = padded_n(n);
  if (((uintptr_t)ws & 255) || ws_bytes < (size_t)(6 * np * CAP)) return GPTAQ_EWORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  const Operands o = operands_at(ws, np, CAP, false);
  auto products = [&](int64_t cp) { return launch_products(o, np, cp, n, H, dXXT, ldh, dxxt_upper, ws, ws_bytes, s); };
  int64_t done = 0, pend = *pending;
  while (done < tokens) {
    const int64_t take = tokens - done < CAP - pend ? tokens - done : CAP - pend, cp = round_up(take, 64);
    if (const int rc = launch_split(o, X + done * ldx, Xtilde + done * ldx, ldx, take, n, np, pend / 64, nullptr, s)) return rc;
    done += take;
    pend += cp;                                    // (only the chunk that comes with flush may be ragged: it is the last)
    if (pend >= CAP) {
      hipError_t e = products(CAP);
      if (e != hipSuccess) { set_last_hip_error(e); return GPTAQ_ELAUNCH; }
      pend = 0;
    }
  }
  if (flush && pend > 0) {
    hipError_t e = products(pend);
    if (e != hipSuccess) { set_last_hip_error(e); return GPTAQ_ELAUNCH; }
    pend = 0;
  }
  *pending = pend;
  return GPTAQ_OK;
}

extern "C" int gptaq_accumulate_staged(const uint16_t* X, const uint16_t* Xtilde, int64_t tokens, int64_t n, int64_t ldx,
                                       float* H, float* dXXT, int64_t ldh, void* ws, size_t ws_bytes, int64_t* pending,
                                       int flush, void* stream) {
  return accumulate_staged_impl(X, Xtilde, tokens, n, ldx, H, dXXT, ldh, false, ws, ws_bytes, pending, flush, stream);
}

extern "C" int gptaq_accumulate_staged_upper(const uint16_t* X, const uint16_t* Xtilde, int64_t tokens, int64_t n,
                                             int64_t ldx, float* H, float* dXXT, int64_t ldh, void* ws, size_t ws_bytes,
                                             int64_t* pending, int flush, void* stream) {
  return accumulate_staged_impl(X, Xtilde, tokens, n, ldx, H, dXXT, ldh, true, ws, ws_bytes, pending, flush, stream);
}

extern "C" int gptaq_symmetrize(float* H, int64_t n, int64_t ldh, void* stream) {
  if (!H) return GPTAQ_ENULL;
  if (n <= 0 || ldh < n || n > (1 << 20)) return GPTAQ_EDIM;
  const unsigned g = (unsigned)((n + 31) / 32);
  hipLaunchKernelGGL(symmetrize_kernel, dim3(g, g), dim3(32, 32), 0, (hipStream_t)stream, H, (int)n, ldh);
  GPTAQ_LAUNCH_CHECK();
  return GPTAQ_OK;
}
