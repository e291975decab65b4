// Which matrices the column loop takes as two row halves.  Host code, without HIP, so that a compiler without it can check the rule.
#pragma once
#include <stdint.h>

namespace gptaq {

// How many of its m rows the first half takes where a matrix of nsb super-blocks is quantised as two row halves (on two streams, so that
// each half's super-block kernel runs beside the other's far update); 0 where it is not.  A multiple of the GEMM's row tile, so that the
// halves' padded rows of the -E / V buffers do not overlap, and less than m: up to 256 rows there is no second half.
// Instead, 1025 to 4096 rows of three super-blocks or more go through as two chains (quantize_layer_sb), others as one.  Both measured, in
// their order, us, W4 g128, both terms.  One chain / halves, many rows: 3072 columns: 7168 rows 677 / 655, 8192 703 / 703, 9216 848 / 763; 4096:
// 4352 927 / 866, 6144 1070 / 983; 5120: 5120 1377 / 1350; few: 8192: 512 1593 / 1689, 1024 1632 / 1713; 9216: 1024 1882 / 1937; 10240: 820 2126 /
// 2166, 1024 2176 / 2170; 11008: 512 2262 / 2307, 745 2344 / 2338, 900 2454 / 2347, 1024 2473 / 2386; 14336: 400 3047 / 3061, 586 3203 / 3123,
// 640 3152 / 3195, 700 3307 / 3233, 1024 3481 / 3313; also where the second half is much the shorter one: 16384: 384 3501 / 3629, 513 3797 / 3670, 1024
// 4157 / 3974; 28672: 293 7407 / 7347, 512 7862 / 7695, 1024 9999 / 9412; 53248: 257 18379 / 18018, 512 20276 / 19881.
// Two chains / halves: 4096: 4096 772 / 836; 5120: 4096 1103 / 1205; 5248: 1366 1030 / 1021, 2048 1040 / 1064, 3584 1172 / 1243; 5504: 4096 1361 / 1353;
// 6144: 1366 1189 / 1184, 2048 1245 / 1300, 4096 1478 / 1621; 8192: 1100 1696 / 1687, 1536 1766 / 1810, 2048 1799 / 1832, 3584 2199 / 2288, 4096 2291 /
// 2435 (with the clip search 3342 / 3627); 9216: 1100 1978 / 1919, 1536 2076 / 2014, 1792 2104 / 2262; 10240: 1536 2388 / 2246, 1792 2428 / 2558;
// 11008: 1100 2508 / 2393, 1536 2681 / 2538, 1664 2700 / 2765, 2048 2778 / 2857, 3584 3523 / 3632, 4096 3736 / 3801; 14336: 1536 3959 / 3813, 1664 3840 / 3993,
// 4096 5832 / 5890; 16384: 1280 4557 / 4462, 1536 4722 / 4474, 2048 4859 / 5179; 28672: 1536 11243 / 11215, 2048 12167 / 12840; 53248: 1100 28477 / 27924,
// 1536 32279 / 33667.
// (Single terms and the clip search keep the line from 10240 rows on.)
inline int64_t first_row_half(int64_t m, int64_t nsb, int terms, bool clip) {
  const int64_t first = (m + 511) / 512 * 256;
  auto halves = [&]() {
    if (terms == 0 || nsb < 2) return false;
    if (m >= 10240) return true;
    if (terms != 3 || clip || nsb == 2) return false;
    if (nsb == 3) return m >= 8192;
    if (m > 1536) return m > 4096;
    return m > 1024 ? nsb >= 9 : nsb >= 11 && m * nsb >= 8192;
  };
  return halves() && first < m ? first : 0;
}

}  // namespace gptaq
