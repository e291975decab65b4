// Internal declarations shared by the translation units of libgptaq (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <mutex>
#include <vector>
#include "../../include/gptaq.h"

namespace gptaq {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) __bf16 bf16x16;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kGemmBK = 32;          // bf16 elements per k-tile of the MFMA GEMM

inline int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

// One term of a GEMM: up to two left and two right bf16 operands (hi, lo) sharing one layout.
// Element (row, k) of an operand sits at base + row * ld + (k / 32) * kt + k % 32:  ld = K, kt = 32
// for a plain row-major K-contiguous matrix;  ld = 32, kt = rows * 32 for the k-tile-major layout, in
// which the 32-wide k-tile of a block of rows is one contiguous run (no power-of-two row stride, so a
// tile's lines spread over all memory channels).
struct GemmTerm {
  const uint16_t* L[2];
  const uint16_t* R[2];
  int64_t ldl, ldr;
  int64_t ktl, ktr;
};

// Kind 3: L[0] = hi and R[0] = X as above, k-tile-major.  Of lo, the remainder of hi, few entries are not zero.  It is taken by 32 x 32 blocks
// (32 columns of the caller's X, one k-tile) in one or two v_smfmac_f32_32x32x32_bf16, whose left operand is two values of every four
// tokens and 16 bits that say which: 16 bytes for tokens 0 .. 15 of a row and 16 for 16 .. 31.
// Sparse block, no four tokens of a row hold more than two values that are not zero: lo1 has these values, and positions say where they sit.
// Dense block: lo1 has the values of tokens 0 and 1 of every four, lo2 those of 2 and 3, positions are the same for all.
// By blocks (lo_rows = 0): L[1] is lo1, 32 bytes a row and k-tile.  R[1] has as many bytes again, 4 KB for the four blocks of 128 rows:
// four heads of 16 bytes, four position fields of 128, four tails of 880.  A sparse block has kSparseMark in its head and 4 bytes a row in
// its position field, and its tail is not used; head, position field and tail of a dense one, one after the other, are lo2.
// By rows (lo_rows = 1), for rows in another order than the columns of X, so that the two kinds lie among each other: L[1] is 64
// bytes a row and k-tile, lo1 and then lo2; of a sparse block's rows each 16 bytes of lo2 are kRowMark with the positions in its low half, and zeros.
// The marks are NaNs that no remainder is: those that arithmetic makes are quiet.
constexpr uint32_t kSparseMark = 0x7f817f81u, kRowMark = 0x7f810000u;
constexpr int kMaxRemainderK = 32768;      // K of a problem of kind 3 (a multiple of 64)

// C (+)= sum_t sum_pairs L R^T.  kind 0: L0 R0.  kind 1: L0 R0 + L1 R0 (two left operands share the
// right one).  kind 2: L0 R0 + L0 R1 + L1 R0 (hi/lo split of both sides, lo*lo dropped).  kind 3: (hi + lo) X^T (one term; see above).
// Operand buffers are zero-padded to whole tiles in rows and to a multiple of kGemmBK in K, so the
// main loop needs no bounds checks; stores are bounded by M and N.
struct GemmProblem {
  float* C;
  int64_t ldc;
  int32_t M, N, K;       // K per term (multiple of kGemmBK)
  int32_t tiles_m, tiles_n;
  int32_t kind, nterm;
  int32_t tile_mode;     // 0: all tiles; 1: tiles entirely below the diagonal do no work (but store);
                         // 2: square problem, only tiles with tile column >= tile row are scheduled
  int32_t k_mode;        // 0: all k; 1: k >= first column of the tile; 2: tile row0 <= k < tile col end
  int32_t store_mode;    // 0: C += acc; 1: C = acc; 2: C = acc where col > row, else 0; 3: as 2, in out_hi and out_lo instead of C
  int32_t deal;          // how the tile list is shared out to the 8 XCDs: 0: one contiguous run each (tiles of equal
                         // length); 1: dealt four tiles at a time (tile lengths that vary along the list: k_mode 1, 2)
  int32_t split;         // > 1 (128-tiles, k_mode 0, store_mode 0): K in so many parts, each summed by workgroups of its own into
  float* partial;        // `partial` (tiles * split * 128 * 128 floats), and added to C by a second kernel; 0 counts as 1
  int32_t quartered;     // (256-tiles of kind 0 in a batch of kind 3, second problem) so many of its last tiles are taken as four of 128 x 128
  int32_t lo_rows;       // kind 3: how lo lies (see above)
  uint16_t *out_hi, *out_lo;      // store_mode 3: k-tile-major with ldc rows, the tiles that have work
  GemmTerm term[2];
};

struct GemmBatch {
  int32_t nprob;
  int32_t tile;          // 128 or 256 (square block tile)
  int32_t ntiles[2];     // filled by launch_gemm
  int32_t diag_wgs;      // filled by launch_gemm: workgroups that sum the diagonal of a split upper-triangular second problem in one part
  int32_t max_wgs;       // 0: one workgroup per tile; else at most this many workgroups, each taking several tiles
  GemmProblem p[2];
};

// Enqueue the batch; problems are scheduled in order (put the heavier one first).
hipError_t launch_gemm(const GemmBatch& b, hipStream_t s);
// The same for the sums of a narrow input: kind 1 first, kind 0 of the upper triangle second (tiles_m and tiles_n are filled in).
hipError_t launch_narrow_sums(const GemmBatch& b, hipStream_t s);
// Row padding the GEMM expects from an operand with `rows` logical rows.
inline int gemm_tile_for(int64_t M, int64_t N) {
  // 256 x 256 tiles move the fewest bytes per flop but one workgroup fills a CU; use them only when they
  // still give every CU a tile, otherwise 128 x 128 tiles (two workgroups per CU).
  const int64_t t256 = ((M + 255) / 256) * ((N + 255) / 256);
  return (M >= 1024 && N >= 1024 && t256 >= 224) ? 256 : 128;
}

// fp64-grade rank-k products through digit-sliced int8 MFMA (gemm_i8s.h).  A sliced operand holds
// kI8Planes digit planes of rows_pad x kI8MaxK signed bytes (rows_pad a multiple of 128; rows and k beyond the
// source are zero) and one power-of-two scale (its exponent) per row.
constexpr int kI8Planes = 6;
constexpr int kI8MaxK = 256;
struct I8Operand {
  uint8_t* planes;
  int32_t* scale;
  int64_t rows_pad;
  __host__ __device__ int64_t chunk_stride() const { return rows_pad * 32; }
  __host__ __device__ int64_t plane_stride() const { return rows_pad * kI8MaxK; }
  static size_t plane_bytes(int64_t rows_pad) { return (size_t)kI8Planes * rows_pad * kI8MaxK; }
};
struct I8Gemm {
  const uint8_t* A; int64_t a_plane, a_chunk; const int32_t* sa;
  const uint8_t* B; int64_t b_plane, b_chunk; const int32_t* sb;
  double* C; int64_t ldc;
  int32_t M, N, nchunk, beta, upper_only, tiles_m, tiles_n, tile0, ntile;      // tiles tile0 .. tile0 + ntile - 1 of the list
  double alpha;
};
// The fp64 part of the factor sweep, one outer block of kFactorBlock columns [o0, o0 + kFactorBlock) at a time (o0 a multiple of
// it; the block may reach past n).  V holds the block's factor as 16 x 16 tiles, (k, a) at (16 k + a) * 256 doubles; T the second
// half's own block after the first half's update, as tiles (a, b), a >= b, at (a (a + 1) / 2 + b) * 256.
constexpr int kFactorBlock = 256;
constexpr size_t kFactorTileBytes = (size_t)kFactorBlock * kFactorBlock * 8, kHalfTileBytes = (size_t)36 * 256 * 8;
constexpr size_t kBlockSyncBytes = 768;
struct BlockFactor {
  const double* F; int64_t ldf; int n, o0;
  int32_t* info;                     // set to 1 + index of the first pivot that is not positive, unless set already
  double *V, *T;
  int32_t* sync;                     // kBlockSyncBytes, zeros
};
struct BlockPanel {
  I8Operand Vs;                      // out: digits of V_I,OB, rows I = 0 .. o0 - 1
  I8Operand Ucol;                    // out: digits of the columns of U_OB,OB
  double* Uob;                       // out: U_OB,OB, kFactorBlock x kFactorBlock by columns, zeros below the diagonal;
  double* Uout;                      // its upper part also to F_OB,OB
};

// Column loop + in-super-block updates of a whole super-block in one launch (quantize_sb.hip).
constexpr int kSbCols = 1024;       // columns per super-block
// What the kernel reads of U and P: places for every super-block of a layer (layout: near_operands_kernel).
struct SbNear {
  uint16_t* left;                    // U hi, U lo, P hi, P lo, `stride` elements apart: kSbCols * kSbCols bf16 per super-block each
  int64_t stride;
  float* diag;                       // kSbCols / 16 * 512 floats per super-block
  __host__ SbNear at(int sb) const {
    SbNear o = *this;
    o.left += (int64_t)sb * kSbCols * kSbCols;
    o.diag += (int64_t)sb * (kSbCols / 16) * 512;
    return o;
  }
};
struct SbArgs {
  float* W; int64_t ldw; int m, n;
  int sb0, sbw;                      // first column and width (<= kSbCols) of the super-block
  SbNear near;                       // of this super-block
  float maxq; int group, sym, G, terms;
  float* scales; float* zeros; uint8_t* codes;
  uint16_t* EV;                      // -E hi, -E lo, V hi, V lo of the super-block, `evstride` elements apart, k-tile-major (NULL: not
  int64_t evstride, evkt;            // wanted): element (row, k) at (k / 32) * evkt + 32 * row + k % 32
  int clip_grid, clip_steps;         // clip-range search of every group (0 steps: plain min-max; groups only)
  int fast_rows;                     // rows of W and of codes may be stored 16 bytes at a time
};
// Operands of super-blocks first .. first + count - 1, to the first `count` places of o.
hipError_t launch_near_operands(const float* U, const float* P, int64_t ldh, int n, int first, int count, const SbNear& o, hipStream_t s);
hipError_t launch_quant_sb(const SbArgs& a, hipStream_t s);

void set_last_hip_error(hipError_t e);

// Helper stream of the library: entry points that run two chains of kernels side by side (the far updates of
// gptaq_quantize_layer, its row halves) put one chain on the caller's stream and the other on this
// stream, tied together with events on both ends, so that to the caller the call is still one asynchronous
// operation on its own stream.  One stream (default priority) and one growing pool of events per device, created on
// first use and kept until the process ends.  The mutex serialises the host threads that enqueue through it.
struct SideStream {
  hipStream_t stream = nullptr;
  std::vector<hipEvent_t> events;
};
std::mutex& side_stream_mutex();
// The current device's helper stream with at least `nevents` events; nullptr on failure (call with the mutex held).
SideStream* side_stream(int nevents);

// Raises a kernel's dynamic LDS limit exactly once per process, whichever host thread comes first; every caller
// gets the result of that one attempt.
struct LdsLimitOnce {
  std::once_flag once;
  hipError_t result = hipSuccess;
  hipError_t ensure(const void* kernel, int bytes) {
    std::call_once(once, [&] { result = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); });
    return result;
  }
};

// Optional per-kernel timing with HIP events (gptaq_profile_* in the public header).
enum ProfTag { kProfAccumGemm = 0, kProfAccumSplit = 1, kProfFactor = 2, kProfPGemm = 3, kProfColumnLoop = 4,
               kProfTrailGemm = 5, kProfTrailSplit = 6, kProfTags = 7, kProfNone = -1 };
bool prof_enabled(int tag);
void prof_mark(int tag, hipStream_t s, bool begin);
struct ProfScope {
  int tag; hipStream_t s; bool on;
  ProfScope(int t, hipStream_t st) : tag(t), s(st), on(t != kProfNone && prof_enabled(t)) { if (on) prof_mark(tag, s, true); }
  ~ProfScope() { if (on) prof_mark(tag, s, false); }
};

#define GPTAQ_LAUNCH_CHECK()                                   \
  do {                                                         \
    hipError_t e__ = hipGetLastError();                        \
    if (e__ != hipSuccess) { set_last_hip_error(e__); return GPTAQ_ELAUNCH; } \
  } while (0)

}  // namespace gptaq
