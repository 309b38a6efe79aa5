// Which fp32 MLPs' first hidden layer goes by column strips (kernels_mlp_strip.hip), over how many ranges of the weights' rows, and
// the byte offsets that its lanes form.  Plain host code, and callable from the kernel where it is constexpr.
#pragma once
#include <cstdint>

namespace ols {

constexpr int kStripRows = 64, kStripCols = 128;       // weight rows of a tile, columns of a strip
constexpr unsigned kStripNowhere = 0x80000000u;        // a lane without a column or a sample's rows starts here: zeros, and nothing is stored

// samples that a workgroup has places for (zeros past the batch)
constexpr int strip_samples(int B) { return B <= 64 ? 64 : 128; }

// Byte offset of row `row` of a lane whose column's offset (or kStripNowhere) is `lane`, in a matrix with `row_bytes` per row.
constexpr unsigned strip_offset(unsigned lane, unsigned row, unsigned row_bytes) { return lane + row * row_bytes; }

// The offsets are 32 bits, and lanes add rows that do not exist to them, also to kStripNowhere: rows of a last tile past the weights,
// samples past the batch.  With every operand, rounded up to whole tiles of rows and to strip_samples, below 2^31 bytes no sum passes 2^32
// (where it would be a place in the matrix again), and all of them lie past the operand's end.  The limit is gemm_split_fits's, whose
// forward GEMM such a layer takes.  B samples, layer K -> N.
inline bool mlp_strip_offsets_fit(int B, int N, int K) {
    const int64_t most = ((int64_t)1 << 29) - 65536, rows = ((int64_t)K + kStripRows - 1) / kStripRows * kStripRows, samples = strip_samples(B);
    return rows * N < most && samples * K < most && samples * N < most;
}

// The rule.  A workgroup takes a compute unit; its time is its tiles and about one and a half more for its start and end.  Ranges
// are chosen for the fewest such times, within one round of the compute units if half of it is work (0.6 where that is more than
// eight tiles; columns that a last strip does not have count as none), else over several rounds if 0.72 of them is: a last round that is nearly empty costs more than the saved
// pass over the weights.  Contractions of up to 1024 stay in one range.  Two rounds, us without / with it.  One round, share: 0.51: 2
// x (2544-1364-10, batch 92) 337 / 302;  0.65: 15 x (2368-352-448-10, 108) 635 / 534;  0.68: 3 x (2488-1188-10, 48) 600 / 480;  0.86:
// 64 x (2164-240-10, 48) 767 / 603;  0.45 (not taken): 55 x (2660-144-10, 28) 306 / 340.  Several rounds: 0.72: 15 x (1664-1536-480-10,
// 112) 1566 / 1496, 52 x (1524-1800-10, 20) 2832 / 2903;  0.73: 21 x (1492-1060-10, 48) 845 / 743;  0.82: 33 x (1868-1704-428-2016-5, 16)
// 5387 / 5034;  not taken: 0.62: 22 x (1888-692-10, 96) 1730 / 2018;  0.69: 18 x (1312-1024-10, 88) 1338 / 1432 (0.53 in one round: the same), 10 x (1952-1248-96-10,
// 16) 1196 / 1040.  Short contractions of more than 64 samples, whose tiles take longer, have to fill 0.56 of the one round: below it
// 23 x (1492-404-2, 76) tau 1 0.90 times as fast, 32 x (1224-300-13, 124) tau 1 0.94, 44 x (296-492-6, 96) 0.97, 31 x (844-604-5, 108) 1.04,
// but 9 x (2228-380-8, 124) 1.27, 2 x (1908-1512-9, 124) 1.23.
// Those figures are for ols_run_steps.  Callers that drive the steps one by one take the same two kernels without the product ahead,
// for the same bits: 110 shapes 1.05 times as fast as without strips in the geometric mean, 0.90 the least (27 x (2400-184-11, 24)), where
// ols_run_steps is 1.21 and 1.15 times as fast.
inline bool mlp_strip_plan(int groups, int B, int N, int K, int most_ranges, int* ranges) {
    if (B > 128 || N % 4 || K % 4 || !mlp_strip_offsets_fit(B, N, K)) return false;
    const int64_t strips = (int64_t)groups * ((N + kStripCols - 1) / kStripCols), tiles = (K + kStripRows - 1) / kStripRows;
    if (strips > (1 << 20)) return false;
    const double work = (double)groups * N / kStripCols * (double)tiles / 256.0;
    double one = 0.0, several = 0.0;
    int r_one = 1, r_several = 1;
    for (int r = 1; r <= (K > 1024 ? most_ranges : 1) && (r == 1 || tiles / r >= 3); ++r) {
        const int64_t per = (tiles + r - 1) / r, used = (tiles + per - 1) / per, rounds = (strips * used + 255) / 256;
        const double share = work / ((double)rounds * ((double)per + 1.5));
        if (rounds == 1 && share > one) { one = share; r_one = (int)used; }
        if (rounds > 1 && share > several) { several = share; r_several = (int)used; }
    }
    const bool fits_one = one >= (work > 8.0 ? 0.6 : B > 64 && K < 1600 ? 0.56 : 0.5);
    *ranges = fits_one ? r_one : r_several;
    return fits_one || several >= 0.72;
}
inline int mlp_strip_range_rows(int K, int ranges) { return ((K + kStripRows - 1) / kStripRows + ranges - 1) / ranges * kStripRows; }

// The ranges of a launch without the next product, whose bits do not depend on them: the caller drives the steps one by one.  More
// rounds than one end more evenly in four ranges: us per launch 64 x (3072 x 1024, batch 64) 598 / 590, 64 x (756 x 1264, 24) 211 / 199.  A
// launch that only writes the gradient holds two workgroups per compute unit and takes eight: steps of 63 x (2752-252-5, 16) 257 / 237,
// 11 x (2628-1108-5, 92) 294 / 253, 40 x (1900-688-10, 32) 319 / 299, 45 x (1556-512-2, 64) 238 / 218.
inline int mlp_strip_alone_ranges(int groups, int N, int K, int ranges, bool update) {
    const int64_t strips = (int64_t)groups * ((N + kStripCols - 1) / kStripCols), tiles = (K + kStripRows - 1) / kStripRows;
    if (!update) return (int)(tiles < 8 ? tiles : 8);
    return strips > 256 && ranges < 4 && tiles >= 12 ? 4 : ranges;
}

}  // namespace ols
