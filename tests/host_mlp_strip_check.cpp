// Host check of the strip kernel's byte offsets (csrc/mlp_strip_plan.h).  For every layer that the rule takes, near the largest
// operands that it may: what its lanes form for rows and samples that exist is their place, and what they form for those that do
// not -- rows of the last tile past the weights, samples past the batch, lanes without a column -- lies past the operand's end
// and does not wrap.  Built with the host compiler by tests/test_mlp_strip_plan_cpu.py; prints the number of mismatches -- or, with
// arguments "workers batch columns rows" for any number of first layers, over how many ranges each goes by column strips.
#include "gemm_f32_plan.h"

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

using namespace ols;

static long bad = 0, taken = 0;

// rows first .. last of an operand with `rows` rows of `cols` columns, as the lanes of the last column and of none reach them
static void operand(const char* what, int64_t first, int64_t last, int64_t rows, int64_t cols, int B, int N, int K) {
    const uint64_t bytes = 4ull * rows * cols;
    const unsigned row_bytes = 4u * (unsigned)cols;
    for (int64_t r = first; r <= last; ++r) {
        const uint64_t place = 4ull * (r * cols + cols - 4);
        const unsigned got = strip_offset(4u * (unsigned)(cols - 4), (unsigned)r, row_bytes);
        const unsigned idle = strip_offset(kStripNowhere, (unsigned)r, row_bytes);
        const bool ok = (r < rows ? got == place : got >= bytes) && idle >= bytes;
        if (!ok && bad++ < 5) std::printf("%s row %ld of %ld x %ld (batch %d, %d -> %d): %u and %u of %lu bytes\n", what, (long)r, (long)rows, (long)cols, B, K, N, got, idle, (unsigned long)bytes);
    }
}

static void check(int B, int N, int K) {
    int ranges;
    bool any = false;
    for (int groups : {1, 2, 3, 5, 8, 64}) any = any || mlp_strip_plan(groups, B, N, K, 8, &ranges);
    if (!any) return;
    ++taken;
    const int64_t tiles = ((int64_t)K + kStripRows - 1) / kStripRows;
    operand("weights", (tiles - 1) * kStripRows, tiles * kStripRows - 1, K, N, B, N, K);
    operand("batch", 0, strip_samples(B) - 1, B, K, B, N, K);
    operand("delta", 0, strip_samples(B) - 1, B, N, B, N, K);
}

int main(int argc, char** argv) {
    if (argc > 1) {
        for (int i = 1; i + 3 < argc; i += 4) std::printf("%d\n", mlp_first_layer_strips(std::atoi(argv[i]), std::atoi(argv[i + 1]), std::atoi(argv[i + 2]), std::atoi(argv[i + 3]), false));
        return 0;
    }
    check(32, 9996, 53700);    // 2 x (53700-9996-10): 31 KiB per row, 60 rows of the last tile do not exist
    check(32, 3040, 176580);
    check(64, 512, 3072);
    uint64_t rng = 0x9E3779B97F4A7C15ull;
    auto draw = [&](uint64_t n) { rng = rng * 6364136223846793005ull + 1442695040888963407ull; return (int64_t)((rng >> 20) % n); };
    for (int t = 0; t < 20000; ++t) {   // layers around 2^29 weights, and batches around 2^29 elements
        const int B = 4 * (1 + (int)draw(32));
        const int64_t N = 4 * (1 + draw(t % 3 == 0 ? 25 : 40000));
        int64_t K = (((int64_t)1 << 29) - draw(1 << 20)) / (t % 3 == 0 ? B * (1 + draw(3)) : N);
        K = K / 4 * 4;
        if (K >= 4 && K < ((int64_t)1 << 31) - 64 && N <= INT32_MAX) check(B, (int)N, (int)K);
    }
    std::printf("%ld layers, %ld mismatches\n", taken, bad);
    return bad != 0 || taken < 1000;
}
