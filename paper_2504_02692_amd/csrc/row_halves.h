// Which matrices the column loop takes as two row halves.  Host code, without HIP, so that a compiler without it can check the rule.
#pragma once
#include <stdint.h>

namespace gptaq {

// How many of its m rows the first half takes where a matrix of nsb super-blocks is quantised as two row halves (on two streams, so that
// each half's super-block kernel runs beside the other's far update); 0 where it is not.  A multiple of the GEMM's row tile, so that the
// halves' padded rows of the -E / V buffers do not overlap, and less than m: up to 256 rows there is no second half.
// Instead, up to 4096 rows go through as two chains (quantize_layer_sb) and more as one.  Both measured, in their order, ms, W4 g128,
// both terms: 3072 columns: 7168 rows 0.69 / 0.69, 8192 0.74 / 0.73, 9216 0.90 / 0.79; 4096: 4096 0.83 / 0.86, 4352 0.93 / 0.88, 6144
// 1.15 / 1.00, 8192 1.35 / 1.26; 5120: 4096 1.18 / 1.26, 5120 1.47 / 1.39; from six super-blocks on the far updates set the pace: 5248:
// 1366 1.13 / 1.07, 2048 1.14 / 1.10, 3584 1.27 / 1.27; 5504: 4096 1.54 / 1.38, 6144 1.96 / 1.65; 6144: 1366 1.29 / 1.22, 2048 1.35 / 1.34,
// 3584 1.66 / 1.51; 8192: 1024 1.85 / 1.75, 2048 2.00 / 1.99, 3584 2.44 / 2.32, 6144 3.55 / 2.94; 11008: 745 2.55 / 2.39, 1024 2.71 / 2.43,
// 2048 3.04 / 2.88, 3584 3.76 / 3.65, 4096 3.97 / 3.76; 14336: 640 3.35 / 3.20, 4096 6.11 / 5.74; also where the second half is much the
// shorter one: 16384: 513 3.93 / 3.70; 28672: 293 7.96 / 7.37, 512 8.40 / 7.72; 53248: 257 18.9 / 18.0, 512 21.2 / 19.9.
// Not there: 3072 rows of 6144 columns 1.45 / 1.53, of 11008 3.49 / 3.60; 1024 of 6144 1.24 / 1.23; and with the clip search, where the
// super-block kernel sets the pace again, 4096 x 8192 3.54 / 3.72 (it and single terms keep the line from 10240 rows on).
inline int64_t first_row_half(int64_t m, int64_t nsb, int terms, bool clip) {
  const int64_t first = (m + 511) / 512 * 256;
  auto halves = [&]() {
    if (terms == 0 || nsb < 2) return false;
    if (m >= 10240) return true;
    if (terms != 3 || clip || nsb == 2) return false;
    if (nsb == 3) return m >= 8192;
    if (nsb < 6) return m > 4096;
    return m >= 3584 || (m <= 2048 && m * nsb >= 8192);
  };
  return halves() && first < m ? first : 0;
}

}  // namespace gptaq
