// Grouped fp32 GEMMs of small launches: forward and back-propagated delta of the per-worker MLPs (whose gradients are the
// g_i of Section 2, arXiv 2002.09539) where 64 x 64 tiles are too few for the chip, so that a launch's time is one tile's chain
// of K slices -- load, LDS, barrier, fragments -- and not throughput.
//
//   FWD  C[M][N] = relu(A[M][K] W[K][N] + bias[N])
//   DA   C[M][N] = (A[M][K] B[N][K]^T) * [mask > 0]
//
// A workgroup owns a 32 x 16 tile (32 x 32 in larger launches); its four wavefronts share out the contraction (wavefront w
// takes steps w, w + 4, .. of 16 indices) and load their MFMA fragments (v_mfma_f32_16x16x4_f32) straight from memory: no LDS
// and no barrier before the wavefronts' sums meet in LDS, in wavefront order.  Lane l of a fragment holds indices
// 4 (l / 16) .. + 3 of its step, one per MFMA, for both operands: 16-byte loads where the contraction index is contiguous, four
// dwords of 64 contiguous bytes per 16 lanes where it is not.  Buffer descriptors return zeros past the operands' ends.  How many
// steps, up to eight, are requested together is a template parameter, so that no load is issued for nothing (with twelve
// always requested, 5 x (36 x 124 x 300) took 8.0 us instead of 4.0).  In the forward kernels they are one round trip, and the
// registers grow with their number (24 to 114 and the sums).  Not so in the delta's: the compiler moves the loads of a step
// between the products of the steps before it, so that about two steps are in flight whatever the number (36 registers from
// three on) and a wavefront waits once per step.  The rules below and the following figures were measured on these kernels as
// they are; so was that eight or sixteen wavefronts per tile are no faster on any of 70 shapes by more than 8 % and slower on
// most.
//
// us per launch, 64 x 64 tiles (forward with the pass that adds their K ranges) / here:
//   workers x (M x N x K)     forward       delta
//   4 x (32 x 96 x 64)        6.2 / 2.8     7.7 / 2.7
//   5 x (36 x 124 x 300)     11.8 / 4.0    12.9 / 3.5
//   5 x (36 x 300 x 788)     11.6 / 6.8    23.9 / 6.1
//   11 x (100 x 312 x 188)    9.0 / 5.3    10.5 / 5.2
//   34 x (60 x 188 x 412)    15.1 / 9.1    16.1 / 10.6
//   6 x (220 x 608 x 604)    28.4 / 19.1   20.7 / 19.9
//   7 x (92 x 824 x 1580)    35.6 / 38.7 (not taken)   43.1 / 41.6
#include "gemm_bf16_tile.h"
#include "gemm_f32_plan.h"
#include "ols_internal.h"

namespace ols {

namespace {

enum { kFwd = 0, kDa = 1, kFwdCast = 2 };   // kFwdCast (bf16): forward from the fp32 batch, see SmallDevB::a32
constexpr int kXcds = 8;
constexpr int kW = 4, kThreads = 64 * kW;          // wavefronts that share a tile's contraction

struct SmallDev {
    const float* a;
    const float* b;
    float* c;
    const float* bias;
    const float* mask;
    int64_t sa, sb, sc, sbias, smask;
    int M, N, K, lda, ldb, ldc;
    int tiles_m, tiles_n, total_tiles, chunk;
};

template <int MODE, int TM, int TN, int S, int CHAINS, bool MORE>
__global__ __launch_bounds__(kThreads) void gemm_f32_small_kernel(SmallDev p) {
    constexpr int BM = 16 * TM, BN = 16 * TN, kOut = BM * BN, kPer = kOut / kThreads;
    __shared__ float red[kW][kOut];
    // a group's tiles stay on one XCD (workgroups are dealt to the XCDs in turn), whose L2 then holds its weights
    const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
    const int tile = xcd * p.chunk + slot;
    if (tile >= p.total_tiles) return;
    const int per_group = p.tiles_m * p.tiles_n, group = tile / per_group;
    const int m0 = tile % per_group / p.tiles_n * BM, n0 = tile % p.tiles_n * BN;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64, l16 = lane % 16, k4 = lane / 16 * 4;

    // the epilogue's inputs come first: output o = thread + u kThreads of the tile lies in block o / 256 (see the accumulators' layout)
    float extra[kPer];
    auto row_of = [&](int o) { return m0 + 16 * (o / 256 / TN) + 4 * (o % 64 / 16) + o % 256 / 64; };
    auto col_of = [&](int o) { return n0 + 16 * (o / 256 % TN) + l16; };
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int o = threadIdx.x + u * kThreads, row = row_of(o), col = col_of(o);
        extra[u] = 0.0f;
        if (row < p.M && col < p.N)
            extra[u] = MODE == kFwd ? p.bias[(int64_t)group * p.sbias + col] : p.mask[(int64_t)group * p.smask + (int64_t)row * p.ldc + col];
    }

    const rsrc_t a_rs = make_rsrc(p.a + (int64_t)group * p.sa, (unsigned)((p.M - 1) * p.lda + p.K) * 4u);
    const rsrc_t b_rs = make_rsrc(p.b + (int64_t)group * p.sb, (unsigned)(MODE == kFwd ? (p.K - 1) * p.ldb + p.N : (p.N - 1) * p.ldb + p.K) * 4u);
    constexpr unsigned kOutside = 0x80000000u;   // beyond every range
    struct Step { f4 a[TM], b[TN]; };
    auto load = [&](Step& r, int step) {
        const int k = 16 * step + k4;
        const bool in = k < p.K;                 // K is a multiple of four
#pragma unroll
        for (int i = 0; i < TM; ++i) {          // (rows past M: beyond the range, or the next row's -- not stored)
            const int row = m0 + 16 * i + l16;
            r.a[i] = __builtin_bit_cast(f4, buf_load(a_rs, in && row < p.M ? 4u * (unsigned)(row * p.lda + k) : kOutside, 0u));
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = n0 + 16 * j + l16;
            if constexpr (MODE == kFwd) {
                const unsigned off = in && col < p.N ? 4u * (unsigned)(k * p.ldb + col) : kOutside;
#pragma unroll
                for (int e = 0; e < 4; ++e) r.b[j][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b_rs, (int)(off + 4u * (unsigned)(e * p.ldb)), 0, 0));
            } else {
                r.b[j] = __builtin_bit_cast(f4, buf_load(b_rs, in && col < p.N ? 4u * (unsigned)(col * p.ldb + k) : kOutside, 0u));
            }
        }
    };
    // A wavefront's steps alternate between CHAINS sums (see small_start)
    f4 acc[CHAINS][TM][TN];
#pragma unroll
    for (int c = 0; c < CHAINS; ++c)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[c][i][j] = f4{0.f, 0.f, 0.f, 0.f};
    auto mfma = [&](const Step& r, int c) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[c][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(r.a[i][e], r.b[j][e], acc[c][i][j], 0, 0, 0);
    };
    const int steps = (p.K + 15) / 16;
    Step r0[S], r1[MORE ? S : 1];
    auto load_trip = [&](Step (&r)[S], int s0) {
#pragma unroll
        for (int t = 0; t < S; ++t) load(r[t], s0 + t * kW);   // (steps past the end: zeros, no traffic)
    };
    auto mfma_trip = [&](const Step (&r)[S]) {
#pragma unroll
        for (int t = 0; t < S; ++t) mfma(r[t], t % CHAINS);
    };
    if constexpr (MORE) {   // the next round trip under way during this one's products
        load_trip(r0, wave);
        for (int s0 = wave; s0 < steps; s0 += 2 * S * kW) {
            load_trip(r1, s0 + S * kW);
            mfma_trip(r0);
            load_trip(r0, s0 + 2 * S * kW);
            mfma_trip(r1);
        }
    } else {
        for (int s0 = wave; s0 < steps; s0 += S * kW) {
            load_trip(r0, s0);
            mfma_trip(r0);
        }
    }
    // Accumulator register r of a lane: row 4 (lane / 16) + r, column lane % 16 of its 16 x 16 block; kept as [block][r][lane]
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[wave][256 * (i * TN + j) + 64 * r + lane] = CHAINS == 1 ? acc[0][i][j][r] : acc[0][i][j][r] + acc[CHAINS - 1][i][j][r];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int o = threadIdx.x + u * kThreads, row = row_of(o), col = col_of(o);
        if (row >= p.M || col >= p.N) continue;
        float v = red[0][o];
#pragma unroll
        for (int w = 1; w < kW; ++w) v += red[w][o];
        v = MODE == kFwd ? fmaxf(v + extra[u], 0.0f) : extra[u] > 0.0f ? v : 0.0f;
        p.c[(int64_t)group * p.sc + (int64_t)row * p.ldc + col] = v;
    }
}

// The same for bf16 operands, fp32 accumulation and bf16 results (v_mfma_f32_16x16x32_bf16: lane l of a fragment holds indices
// 8 (l / 16) .. + 7 of a step of 32).  A tile is 32 x 32; its two column blocks are interleaved (columns 2 (l % 16) and + 1), so
// that the forward pass, whose weights are contiguous along the columns, takes both blocks' fragments from eight dwords of
// neighbouring columns and puts them together with byte permutations, and results leave as pairs.  Up to six steps are
// requested together (a step is ten loads in the forward pass): one round trip in the delta.  In the forward kernels the choice
// between an offset and the end of the range has become a branch per step that waits for all loads before it, so there a
// step is a round trip of its own, up to six in a row; the figures and the rule are of these kernels.
//
// us per launch, 64 x 64 tiles of kernels_gemm_bf16.hip, whose time is their chain of slices through LDS / here:
//   workers x (M x N x K)     forward       delta
//   6 x (24 x 88 x 112)       3.5 / 2.7     3.3 / 2.8
//   6 x (72 x 264 x 520)      6.4 / 4.0     6.0 / 3.7
//   6 x (72 x 520 x 264)      5.1 / 3.9     4.9 / 3.8
//   6 x (72 x 520 x 1032)     9.2 / 6.7     8.2 / 7.4
//   2 x (32 x 168 x 2224)    15.1 / 7.0    12.6 / 8.0
//   24 x (224 x 168 x 120)    4.4 / 3.9     4.4 / 3.8
//
// The first layer's forward GEMM takes the batch as it comes (kFwdCast): a lane loads its eight indices in fp32 and rounds them, and
// the workgroups of a row's first column tile leave the rounded batch for the weight gradient.  The pass that did this alone took
// 4 us and a launch of a small step (6 x (72 x 520 x 1032): 4.0 and 9.3 us then, 13.3 now, so what it saves is the launch).  Two rounds, us, one state / three in turn: 44 x (360-64-12, 184) tau 3 202 -> 180 / 127 -> 119,
// 6 x (264-280-7, 104) tau 3 140 -> 125 / 131 -> 121, 9 x (2032-168-384-3, 72) 216 -> 211 / 174 -> 171, 6 x (1032-520-264-10, 72) 169 -> 167
// (three in turn); none slower.
struct SmallDevB {
    const uint16_t* a;
    const float* a32;        // kFwdCast: A in fp32, in place of a
    uint16_t* a_out;         // kFwdCast: [M][K] per group, the rounded A
    const uint16_t* b;
    uint16_t* c;
    const float* bias;
    const uint16_t* mask;
    int64_t sa, sb, sc, sbias, smask;
    int M, N, K, lda, ldb, ldc;
    int tiles_m, tiles_n, total_tiles, chunk;
};

template <int MODE, int S>
__global__ __launch_bounds__(kThreads) void gemm_bf16_small_kernel(SmallDevB p) {
    constexpr bool FWD = MODE != kDa, CAST = MODE == kFwdCast;
    __shared__ float red[kW][2][2][256];   // [wavefront][row block][column block][register, lane]
    const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
    const int tile = xcd * p.chunk + slot;
    if (tile >= p.total_tiles) return;
    const int per_group = p.tiles_m * p.tiles_n, group = tile / per_group;
    const int m0 = tile % per_group / p.tiles_n * 32, n0 = tile % p.tiles_n * 32;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64, l16 = lane % 16, k8 = lane / 16 * 8;
    const int col = n0 + 2 * l16;   // N is a multiple of eight: the pair is inside or outside together

    // the epilogue's inputs come first: thread t finishes the pairs of row blocks 0 and 1 at (register t / 64, lane t % 64)
    const int row0 = m0 + 4 * (lane / 16) + wave;
    float bias[2] = {0.0f, 0.0f};
    unsigned gate[2] = {0u, 0u};
    if (col < p.N) {
        if constexpr (FWD) {
            bias[0] = p.bias[(int64_t)group * p.sbias + col];
            bias[1] = p.bias[(int64_t)group * p.sbias + col + 1];
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (row0 + 16 * i < p.M) gate[i] = *(const unsigned*)(p.mask + (int64_t)group * p.smask + (int64_t)(row0 + 16 * i) * p.ldc + col);
        }
    }

    const void* A = CAST ? (const void*)(p.a32 + (int64_t)group * p.sa) : (const void*)(p.a + (int64_t)group * p.sa);
    constexpr unsigned kEs = CAST ? 4u : 2u;
    const rsrc_t a_rs = make_rsrc(A, (unsigned)((p.M - 1) * p.lda + p.K) * kEs);
    const rsrc_t b_rs = make_rsrc(p.b + (int64_t)group * p.sb, (unsigned)(FWD ? (p.K - 1) * p.ldb + p.N : (p.N - 1) * p.ldb + p.K) * 2u);
    constexpr unsigned kOutside = 0x80000000u;   // beyond every range
    struct Step { u4 a[CAST ? 4 : 2], b[2]; };   // b: FWD, rows k .. k + 7 of the column pair; DA, eight indices of either column
    auto load = [&](Step& r, int step) {
        const int k = 32 * step + k8;
        const bool in = k < p.K;                 // K is a multiple of eight
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = m0 + 16 * i + l16;
            const unsigned off = in && row < p.M ? kEs * (unsigned)(row * p.lda + k) : kOutside;
            r.a[i] = buf_load(a_rs, off, 0u);
            if constexpr (CAST) r.a[2 + i] = buf_load(a_rs, off, 16u);
        }
        if constexpr (FWD) {
            const unsigned off = in && col < p.N ? 2u * (unsigned)(k * p.ldb + col) : kOutside;
#pragma unroll
            for (int e = 0; e < 8; ++e) r.b[e / 4][e % 4] = __builtin_amdgcn_raw_buffer_load_b32(b_rs, (int)(off + 2u * (unsigned)(e * p.ldb)), 0, 0);
        } else {
#pragma unroll
            for (int j = 0; j < 2; ++j) r.b[j] = buf_load(b_rs, in && col < p.N ? 2u * (unsigned)((col + j) * p.ldb + k) : kOutside, 0u);
        }
    };
    f4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    auto mfma = [&](const Step& r, int step) {
        u4 fa[2], fb[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            fa[i] = r.a[i];
            if constexpr (CAST) {
                const f4 lo = __builtin_bit_cast(f4, r.a[i]), hi = __builtin_bit_cast(f4, r.a[2 + i]);
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    fa[i][w] = bf16_bits_rne(lo[2 * w]) | bf16_bits_rne(lo[2 * w + 1]) << 16;
                    fa[i][2 + w] = bf16_bits_rne(hi[2 * w]) | bf16_bits_rne(hi[2 * w + 1]) << 16;
                }
                const int row = m0 + 16 * i + l16, k = 32 * step + k8;
                if (n0 == 0 && row < p.M && k < p.K) *(u4*)(p.a_out + (int64_t)group * p.M * p.K + (int64_t)row * p.K + k) = fa[i];
            }
        }
        if constexpr (FWD) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const unsigned lo = r.b[w / 2][2 * (w % 2)], hi = r.b[w / 2][2 * (w % 2) + 1];   // rows k + 2 w and k + 2 w + 1
                fb[0][w] = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
                fb[1][w] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
            }
        } else {
            fb[0] = r.b[0];
            fb[1] = r.b[1];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fa[i]), __builtin_bit_cast(bf16x8, fb[j]), acc[i][j], 0, 0, 0);
    };
    const int steps = (p.K + 31) / 32;
    for (int s0 = wave; s0 < steps; s0 += S * kW) {
        Step r[S];
#pragma unroll
        for (int t = 0; t < S; ++t) load(r[t], s0 + t * kW);   // (steps past the end: zeros, no traffic)
#pragma unroll
        for (int t = 0; t < S; ++t) mfma(r[t], s0 + t * kW);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[wave][i][j][64 * r + lane] = acc[i][j][r];
    __syncthreads();
    if (col >= p.N) return;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = row0 + 16 * i;
        if (row >= p.M) continue;
        float v[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            v[j] = red[0][i][j][threadIdx.x];
#pragma unroll
            for (int w = 1; w < kW; ++w) v[j] += red[w][i][j][threadIdx.x];
            if constexpr (FWD) v[j] = fmaxf(v[j] + bias[j], 0.0f);
        }
        unsigned o = __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{v[0], v[1]}, bf16x2));   // to nearest even
        if constexpr (MODE == kDa) {   // a bf16 is positive iff its sign bit is clear and it is not zero
            const unsigned lo = gate[i] & 0xFFFFu, hi = gate[i] >> 16;
            o &= (lo != 0u && lo < 0x8000u ? 0xFFFFu : 0u) | (hi != 0u && hi < 0x8000u ? 0xFFFF0000u : 0u);
        }
        *(unsigned*)(p.c + (int64_t)group * p.sc + (int64_t)row * p.ldc + col) = o;
    }
}

bool aligned16(const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; }

}  // namespace

template <int MODE, int TN>
static void small_start(const SmallDev& p, int steps, hipStream_t s) {
    // as few trips of up to eight steps (requested together) as there have to be, and as short as they then can be
    const int per = (steps + kW - 1) / kW, trips = (per + 7) / 8, S = (per + trips - 1) / trips;
    const unsigned grid = (unsigned)(p.chunk * kXcds);
#define OLS_SMALL(S, CHAINS, MORE) gemm_f32_small_kernel<MODE, 2, TN, S, CHAINS, MORE><<<grid, kThreads, 0, s>>>(p)
    // Round trips one behind the other leave room for more workgroups; with hardly one per compute unit and three trips or more
    // (five to eight steps each) they overlap: forward 3 x (32 x 960 x 1836), 180 tiles, 16.0 -> 12.1, 3 x (40 x 532 x 2236), 204, 18.7 ->
    // 15.1; but 4 x (224 x 124 x 1192), 224 tiles, 8.9 -> 9.8, 17 x (128 x 248 x 1372) 34.3 -> 48.1, and no delta gains.
    //
    // The error of a sum grows with the length of its chain, and the 64 x 64 tiles add forward contractions of 768 indices or more in
    // up to eight K ranges: from there on the four wavefronts have two sums each.  Error of the activations against 64 bits over
    // that of the tiles, 60 shapes: with one sum per wavefront 1.34 (up to 1.40) where they take eight ranges, 1.00 with four,
    // 0.54 with one (like every delta); with two sums 0.96 (up to 1.01) of eight ranges.  The registers of the second sum cost
    // nothing on most shapes (1 % on 4 x (28 x 1924 x 1872)), but 9 % on 6 x (220 x 608 x 604), which does not need it.
    if constexpr (MODE == kFwd && TN == 1) {
        if (trips > 2 && p.total_tiles <= 216) {
            if (S <= 6) OLS_SMALL(6, 2, true);
            else if (S == 7) OLS_SMALL(7, 2, true);
            else OLS_SMALL(8, 2, true);
            return;
        }
    }
    if constexpr (MODE == kFwd) {
        if (p.K >= 768) {   // (twelve steps per wavefront or more: two trips of six to eight at least)
            if (S <= 6) OLS_SMALL(6, 2, false);
            else if (S == 7) OLS_SMALL(7, 2, false);
            else OLS_SMALL(8, 2, false);
            return;
        }
    }
    switch (S) {
        case 1: OLS_SMALL(1, 1, false); break;
        case 2: OLS_SMALL(2, 1, false); break;
        case 3: OLS_SMALL(3, 1, false); break;
        case 4: OLS_SMALL(4, 1, false); break;
        case 5: OLS_SMALL(5, 1, false); break;
        case 6: OLS_SMALL(6, 1, false); break;
        case 7: OLS_SMALL(7, 1, false); break;
        default: OLS_SMALL(8, 1, false); break;
    }
#undef OLS_SMALL
}

static hipError_t small_launch(int mode, const GemmArgs& g, hipStream_t s) {
    const bool fwd = mode == kFwd;
    if (!g.a || !g.b || !g.c || g.groups < 1 || g.M < 1 || g.N < 1 || g.K < 1 || (fwd ? !g.bias : !g.mask)) return hipErrorInvalidValue;
    if (!aligned16(g.a) || !aligned16(g.b) || g.lda % 4 || g.ldb % 4 || g.sa % 4 || g.sb % 4 || g.K % 4 || (fwd && g.N % 4)) return hipErrorInvalidValue;
    if (g.lda < g.K || g.ldb < (fwd ? g.N : g.K) || g.ldc < g.N) return hipErrorInvalidValue;
    SmallDev p = {};
    p.a = (const float*)g.a; p.b = (const float*)g.b; p.c = (float*)g.c; p.bias = g.bias; p.mask = (const float*)g.mask;
    p.sa = g.sa; p.sb = g.sb; p.sc = g.sc; p.sbias = g.sbias; p.smask = g.smask;
    p.M = g.M; p.N = g.N; p.K = g.K; p.lda = g.lda; p.ldb = g.ldb; p.ldc = g.ldc;
    // 32 x 32 tiles (forward only: they halve its many dword loads) once 32 x 16 ones keep the compute units busy for a while:
    // 32 x (24 x 444 x 360), 20,600: 8.8 and 8.0; 4 x (28 x 1924 x 1872), 56,600: 23.0 and 19.3; 4 x (224 x 124 x 1192), 224 tiles: 8.9 and 11.5
    const int steps = (g.K + 15) / 16;
    const int64_t t16 = small_tiles(g.groups, g.M, g.N);
    const bool wide = fwd && t16 >= 256 && t16 * steps >= 16000;
    p.tiles_m = (g.M + 31) / 32;
    p.tiles_n = wide ? (g.N + 31) / 32 : (g.N + 15) / 16;
    const int64_t total = (int64_t)g.groups * p.tiles_m * p.tiles_n;
    if (total > (1 << 30) || !small_offsets((int64_t)g.M * g.lda, (int64_t)(fwd ? g.K : g.N) * g.ldb)) return hipErrorInvalidValue;
    p.total_tiles = (int)total;
    p.chunk = (int)((total + kXcds - 1) / kXcds);
    if (!fwd) small_start<kDa, 1>(p, steps, s);
    else if (wide) small_start<kFwd, 2>(p, steps, s);
    else small_start<kFwd, 1>(p, steps, s);
    return hipGetLastError();
}
hipError_t launch_gemm_small_fwd(const GemmArgs& g, hipStream_t s) { return small_launch(kFwd, g, s); }
hipError_t launch_gemm_small_da(const GemmArgs& g, hipStream_t s) { return small_launch(kDa, g, s); }

// The bf16 rules, from both sides measured on 120 shapes (2 - 61 workers, M 16 - 250, N 64 - 2000, K 64 - 3000) and again on 550, most
// of them near the lines: work in steps of 32 indices of a 32 x 32 tile.
// Forward up to 8,000, and up to 15,000 from K = 640 on and with up to 500 tiles (1.01 - 1.44 times; shorter contractions of that
// size lose: 14 x (168 x 536 x 192), 8,570, 5.5 and 6.0; a step of 3 x 2016-512-1264-4 at batch 208, whose second layer is 13,440
// with K = 512, 2 % of its time; 5 x (240 x 392 x 896), 520 tiles, 10.8 and 11.8).
// Delta up to 7,000 where the tiles are at most 490 for each round of 256 of the 64 x 64 ones (beyond, 0.86 to 1.09 times:
// 16 x (184 x 216 x 320) 7.6 and 8.8, 38 x (64 x 568 x 160) 8.3 and 8.9); from K = 1024 on up to 15,000, with one tile per compute unit
// at most: up to 256 tiles 1.16 - 1.67 times on 80 shapes, with 257 and more 0.83 - 1.13 on 30 (2 x (72 x 1376 x 1088), 258 tiles,
// 10.7 and 12.9).  Of 360 other shapes that the rules take (1.18 and 1.17 times), one forward one loses 5 %, one delta one 8 %
// (5 x (56 x 1736 x 424) 8.6 and 9.1, 3 x (72 x 1304 x 576) 8.7 and 9.5), the rest 3 % at most.
static int64_t small_tiles_bf16(int groups, int M, int N) { return (int64_t)groups * ((M + 31) / 32) * ((N + 31) / 32); }
bool gemm_small_bf16_fits(const GemmArgs& g, bool fwd) {
    const int64_t tiles = small_tiles_bf16(g.groups, g.M, g.N), work = tiles * ((g.K + 31) / 32);
    if (fwd) {
        if (work > (g.K >= 640 && tiles <= 500 ? 15000 : 8000)) return false;
    } else if (g.K >= 1024) {
        if (tiles > 256 || work > 15000) return false;
    } else if (tiles > 490 * tile_rounds(g.groups, g.M, g.N, 1) || work > 7000) {
        return false;
    }
    return small_offsets((int64_t)g.M * g.lda, (int64_t)(fwd ? g.K : g.N) * g.ldb);
}

template <int MODE>
static hipError_t small_bf16(const GemmArgs& g, hipStream_t s) {
    constexpr bool fwd = MODE != kDa, cast = MODE == kFwdCast;
    if (!g.a || !g.b || !g.c || g.groups < 1 || g.M < 1 || g.N < 1 || g.K < 1 || (fwd ? !g.bias : !g.mask)) return hipErrorInvalidValue;
    if (!aligned16(g.a) || !aligned16(g.b) || !aligned16(g.c) || g.lda % 8 || g.ldb % 8 || g.ldc % 8 || g.sa % (cast ? 4 : 8) || g.sb % 8 || g.sc % 8 || g.K % 8 || g.N % 8)
        return hipErrorInvalidValue;
    if (!fwd && (!aligned16(g.mask) || g.smask % 8)) return hipErrorInvalidValue;
    if (g.lda < g.K || g.ldb < (fwd ? g.N : g.K) || g.ldc < g.N) return hipErrorInvalidValue;
    if (!small_offsets((int64_t)g.M * g.lda, (int64_t)(fwd ? g.K : g.N) * g.ldb)) return hipErrorInvalidValue;
    if (cast && (!g.a_rounded || !aligned16(g.a_rounded) || (int64_t)g.M * g.lda >= ((int64_t)1 << 29))) return hipErrorInvalidValue;
    SmallDevB p = {};
    p.a = (const uint16_t*)g.a; p.a32 = (const float*)g.a; p.a_out = (uint16_t*)g.a_rounded; p.b = (const uint16_t*)g.b; p.c = (uint16_t*)g.c; p.bias = g.bias; p.mask = (const uint16_t*)g.mask;
    p.sa = g.sa; p.sb = g.sb; p.sc = g.sc; p.sbias = g.sbias; p.smask = g.smask;
    p.M = g.M; p.N = g.N; p.K = g.K; p.lda = g.lda; p.ldb = g.ldb; p.ldc = g.ldc;
    p.tiles_m = (g.M + 31) / 32;
    p.tiles_n = (g.N + 31) / 32;
    const int64_t total = small_tiles_bf16(g.groups, g.M, g.N);
    if (total > (1 << 30)) return hipErrorInvalidValue;
    p.total_tiles = (int)total;
    p.chunk = (int)((total + kXcds - 1) / kXcds);
    const unsigned grid = (unsigned)(p.chunk * kXcds);
    const int per = ((g.K + 31) / 32 + kW - 1) / kW, trips = (per + 5) / 6;
    switch ((per + trips - 1) / trips) {
        case 1: gemm_bf16_small_kernel<MODE, 1><<<grid, kThreads, 0, s>>>(p); break;
        case 2: gemm_bf16_small_kernel<MODE, 2><<<grid, kThreads, 0, s>>>(p); break;
        case 3: gemm_bf16_small_kernel<MODE, 3><<<grid, kThreads, 0, s>>>(p); break;
        case 4: gemm_bf16_small_kernel<MODE, 4><<<grid, kThreads, 0, s>>>(p); break;
        case 5: gemm_bf16_small_kernel<MODE, 5><<<grid, kThreads, 0, s>>>(p); break;
        default: gemm_bf16_small_kernel<MODE, 6><<<grid, kThreads, 0, s>>>(p); break;
    }
    return hipGetLastError();
}
hipError_t launch_gemm_small_bf16_fwd(const GemmArgs& g, hipStream_t s) { return g.a_rounded ? small_bf16<kFwdCast>(g, s) : small_bf16<kFwd>(g, s); }
hipError_t launch_gemm_small_bf16_da(const GemmArgs& g, hipStream_t s) { return small_bf16<kDa>(g, s); }

}  // namespace ols
