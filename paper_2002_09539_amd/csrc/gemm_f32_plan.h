// Which kernel a GEMM of the fp32 MLPs' hidden layers takes, and over how many K ranges.  Plain host code.
#pragma once
#include <cstdint>

#include "mlp_strip_plan.h"

namespace ols {

// ---- forward and delta GEMMs of small launches: kernels_gemm_small.hip ----
// The rules, from both sides measured on 110 shapes (2 - 64 workers, M 16 - 252, N 64 - 2000, K 64 - 3072) and again on 440, most of
// them near the lines: work in steps of 16 indices of a 32 x 16 tile.  Forward up to 80,000; beyond, 64 x 64 tiles read less; long
// contractions only up to 30,000 (their K ranges spread better: 13 x (40 x 476 x 2612), 128,000, 40.5 and 45.4).  Delta, whose 64 x 64
// tiles have no K ranges, the same without that and up to 160,000 from K = 1024 on (7 x (76 x 1348 x 1396) 63.0 and 54.5;
// 22 x (64 x 536 x 2256), 211,000: 56.9 and 66.4).
// Where the 64 x 64 tiles come close to whole rounds of 256 they are at their best: with more than 1,250 tiles here (1,230 in the
// delta) for each of their rounds, only up to 50,000 (70,000).  Forward 20 x (52 x 236 x 1984) 27.8 and 34.4, 11 x (64 x 412 x 1804) 28.6
// and 34.5, 9 x (100 x 1680 x 300) 21.3 and 23.4, but below 6 x (52 x 644 x 1564), 48,200, 1.21 times as fast; delta
// 6 x (80 x 1160 x 1376) 39.9 and 46.4, 14 x (156 x 364 x 704) 26.9 and 30.6, but 38 x (180 x 492 x 136), 63,600, 1.67 times.  Of 360 other
// shapes that the rules take, the forward ones 1.31 times as fast in the geometric mean and the delta ones 1.70, two forward ones
// lose 3 and 6 % (2 x (84 x 276 x 2536), 18.4 and 19.5).
inline int64_t small_tiles(int groups, int M, int N) { return (int64_t)groups * ((M + 31) / 32) * ((N + 15) / 16); }
inline int64_t tile_rounds(int groups, int M, int N, int ranges) { return ((int64_t)groups * ((M + 63) / 64) * ((N + 63) / 64) * ranges + 255) / 256; }
inline bool small_offsets(int64_t a_elems, int64_t b_elems) { return a_elems < (1 << 28) && b_elems < (1 << 28); }   // 32-bit byte offsets
// `ranges`: the K ranges over which the 64 x 64 tiles would add it; 0: as if they were not at their best
inline bool gemm_small_fwd_fits(int groups, int M, int N, int K, int ranges) {
    const int64_t tiles = small_tiles(groups, M, N), work = tiles * ((K + 15) / 16);
    if (tiles * ranges > 1250 * tile_rounds(groups, M, N, ranges) && work > 50000) return false;   // (never with no ranges)
    return work <= (K <= 2048 ? 80000 : 30000) && small_offsets((int64_t)M * K, (int64_t)K * N);
}
inline bool gemm_small_da_fits(int groups, int M, int N, int K) {
    const int64_t tiles = small_tiles(groups, M, N), work = tiles * ((K + 15) / 16);
    if (tiles > 1230 * tile_rounds(groups, M, N, 1) && work > 70000) return false;
    return work <= (K >= 1024 ? 160000 : 80000) && small_offsets((int64_t)M * K, (int64_t)K * N);
}

// ---- forward GEMMs on the bf16 matrix cores with split operands: kernels_gemm_split.hip ----
inline bool gemm_split_fits(int64_t a_elems, int64_t b_elems) {   // byte offsets of a group's operand below 2^31
    return a_elems < ((int64_t)1 << 29) - 65536 && b_elems < ((int64_t)1 << 29) - 65536;
}

// The rule: 64 x 128 tiles, where they give two workgroups per compute unit, one with long contractions, or half of one over
// four K ranges of at least 512 indices.  Below that the fp32 kernel's smaller tiles fill the chip better: 8 workers x (128 x
// 1024 x 1024) 29 us with it, 28 over four ranges here; 4 x (112 x 120 .. 280 x 1084 .. 120) 13 against 17 us.  With 256 to
// 511 tiles, the fp32 kernel's 64 x 64 tiles against this kernel: 32 x (128 x 512 x 1024) 49 and 47 us, 24 x (192 x 512 x
// 2048) 116 and 107, 40 x (64 x 1024 x 1536) 99 and 95, 16 x (128 x 1024 x 3072) 135 and 135; two K ranges would take 48,
// 105, 92 and 121 us but 64 MB and more of scratch, where these shapes need none.  Contractions are rounded up to groups of
// four slices (128 indices); short ones gain all the same (us per two rounds of two steps, fp32 kernels and these: 64 x (64 x
// 1028 x 36) 367 and 289, 64 x (128 x 2048 x 36) 831 and 632, 64 x (16 x 1024 x 64) 244 and 208, 64 x (64 x 1024 x 132) 399
// and 352).
inline bool gemm_split_fwd_plan(int groups, int M, int N, int K, int* splits) {
    if (N < 128 || !gemm_split_fits((int64_t)M * K, (int64_t)K * N)) return false;
    const int64_t tiles = (int64_t)groups * ((M + 63) / 64) * ((N + 127) / 128);
    *splits = tiles < 256 ? 4 : 1;
    return tiles >= 512 || (tiles >= 256 && K >= 1024) || (tiles >= 128 && K >= 2048);
}

// ---- forward GEMMs: variant (see launch_gemm_f32_fwd) and K ranges; lean: with little scratch ----
// Shape-driven choice for the forward GEMM.  Measured on configuration 2 (M = 128, N = 512, K = 3072,
// 16 groups): every tile shape lands within a few percent once there are several workgroups per compute
// unit, because the matrix pipe idles whenever a wavefront waits at the slice barrier or for its loads
// and only other resident workgroups fill those gaps; so: 64 x 64 tiles, and K ranges until the launch
// has about two workgroups per compute unit.  With the full-tile path, per launch including the pass that
// sums the parts: one K range (256 workgroups) 70.8 us, two 69.1 us, four 71.3 us, eight 82 us; the step as a
// whole 0.1808 / 0.1798 / 0.1828 / 0.194 ms (fewer parts to write and re-read, and the anchor refresh on the
// side stream finds more room beside the smaller launch).
// Where 64 x 64 tiles would give four or more workgroups per compute unit, 64 x 128 tiles (half as many, each
// A slice loaded once for twice the columns) are faster: configuration 5 (M = 64, N = 1024, 64 groups) 232 us
// against 238 us per launch, 0.8428 against 0.8504 ms per step.
// Large launches run on the bf16 matrix cores with split operands (variant 32, kernels_gemm_split.hip: 234 -> 187 us and
// 76 -> 61 us on configurations 5 and 2).  What is left is small: there a K range may be as short as 96 indices (5 workers
// x (36 x 300 x 788): eight ranges 13.8 us, two 17.3), unless the contraction is too short for the second launch that
// adds the ranges up.  Smaller launches still have a kernel without slices and without scratch (variant 33,
// kernels_gemm_small.hip); lean: also where K ranges are a little faster.
inline void gemm_f32_fwd_plan(int groups, int M, int N, int K, bool lean, int* variant, int* splits) {
    *variant = 32;
    if (gemm_split_fwd_plan(groups, M, N, K, splits)) return;
    *variant = 2;
    int64_t tiles = (int64_t)groups * ((M + 63) / 64) * ((N + 63) / 64);
    if (tiles >= 1024 && N >= 128) {
        *variant = 6;
        tiles = (int64_t)groups * ((M + 63) / 64) * ((N + 127) / 128);
    }
    int s = 1;
    while (K >= 512 && tiles * s < 512 && K / (2 * s) >= 96 && s < 8) s *= 2;
    *splits = s;
    if (!gemm_small_fwd_fits(groups, M, N, K, lean && s > 1 ? 0 : s)) return;
    *variant = 33;
    *splits = 1;
}

// Over how many ranges of its weights' rows the first hidden layer (K -> N, B samples) goes by column strips, 0: it does not.
inline int mlp_first_layer_strips(int groups, int B, int N, int K, bool lean) {
    int variant, splits, ranges;
    gemm_f32_fwd_plan(groups, B, N, K, lean, &variant, &splits);
    return variant != 33 && mlp_strip_plan(groups, B, N, K, splits > 1 ? 8 : 1, &ranges) ? ranges : 0;
}

}  // namespace ols
