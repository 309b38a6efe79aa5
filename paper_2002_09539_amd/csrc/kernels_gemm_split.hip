// Forward GEMM of the fp32 MLPs' hidden layers on the bf16 matrix cores, every operand split exactly into three bf16 terms
// while it is staged (split_bf16.h: fp32 accuracy, six bf16 products per fp32 product), grouped over the m workers:
//
//   C[M][N] = relu(A[M][K] W[K][N] + bias[N])
//
// (part of the mini-batch loss whose gradient is the g_i of Section 2, arXiv 2002.09539.)  The fp32 kernels of
// kernels_gemm_f32.hip stay for launches too small to fill the chip with 64 x 128 tiles (gemm_split_fwd_plan), for operands
// past 32-bit offsets, and for the delta and weight-gradient GEMMs.
//
// A slice of 32 contraction indices of each operand goes global -> registers -> split -> LDS.  A's contraction index is
// contiguous: it lies in LDS as rows of 3 x 64 bytes (hi, mid, lo) and is read as 16-byte fragments.  W's row index is
// contiguous: it lies as 32 lines of 3 x 256 bytes and is read with the transpose load.  Both exchange pieces of a row by
// bits of its index, so that every read phase touches the 64 banks once.
//
// What bounds it: 64 workers x (64 x 1024 x 3072) read 0.85 GB (140 us at the rate of the streaming kernels) and are 25.8
// GFLOP, 164 us on the fp32 matrix cores and 62 us as six bf16 products; 16 workers x (128 x 512 x 3072) 0.13 GB and 6.4
// GFLOP.  Measured, us per launch: 234 -> 187 and 76 -> 61 (four K ranges and the pass that adds them included).
// Counters on the first: matrix pipes busy 43 % and vector ALUs (the split) 42 % of the cycles, at an engine clock of 1.78
// GHz.  Tried: 64 x 64 tiles 216 and 65; 128 x 64 305 and 62; 128 x 128 307 and 65; two slices of loads in flight instead
// of four 189 and 62; the instructions of the split dealt out between the products by scheduling groups 194 and 63.  The
// same scheme in the weight-gradient GEMMs, whose contraction is short and whose time is the state's: 64 x 64 tiles 604 and
// 103 against 585 and 102 for the fp32 kernels, 64 x 128 658 and 107: not kept.  In the delta GEMM no difference (12.5
// against 12.7 us on 5 x (36 x 300 x 124)), nor with 64 x 64 tiles in small forward GEMMs.
// Error of a step's gradients against 64 bits (relative 2-norm, median over workers): 1.7e-7 -> 1.4e-7 and 1.9e-7 -> 1.2e-7.
#include "gemm_f32_plan.h"
#include "ols_internal.h"
#include "split_bf16.h"

namespace ols {

namespace {

constexpr int kThreads = 256;
constexpr int kXcds = 8;
constexpr int kBK = 32;
constexpr unsigned kNowhere = 0xFFFFFF00u;   // an offset that the range check answers with zeros

struct GemmSDev {
    const float* a;
    const float* b;
    float* c;
    const float* bias;
    int64_t sa, sb, sc, sbias;
    float* partial;      // split-K: raw partial sums [split][group][M][N]
    int M, N, K, lda, ldb, ldc;
    unsigned a_bytes, b_bytes;   // of a group's operand
    int tiles_m, tiles_n, total_tiles, chunk;
    int splits, k_chunk, groups;
};

// ROWS x 32 slice of an operand.  KC: memory [rows][K]; else memory [K][rows].
// Of the 16 contraction indices of a matrix instruction lane half h takes 8 h + 0 .. 7 -- or, in the strips' order (STRIP), 4 h + 0 .. 3
// and 8 further on: the order in which the accumulators of kernels_mlp_strip.hip hold the weights, so that both leave the same bits.
template <int ROWS, bool KC, bool STRIP>
struct STile {
    static constexpr int kSecond = STRIP ? 8 : 4;   // from the first four of a lane half's indices to the others
    static constexpr int kLine = KC ? 192 : 6 * ROWS;          // bytes of an LDS line: three terms
    static constexpr int kTerm = KC ? 64 : 2 * ROWS;           // bytes between terms
    static constexpr int kBytes = (KC ? ROWS : kBK) * kLine;
    static constexpr int kVecLine = KC ? kBK / 8 : ROWS / 8;   // eight-element vectors per line
    static constexpr int kVecs = ROWS * kBK / 8 / kThreads;    // per lane
    static_assert(ROWS * kBK / 8 % kThreads == 0 && (KC || ROWS == 64 || ROWS == 128), "slice shape");

    struct Lane {
        unsigned off[kVecs][2];   // byte offsets of the vector's two halves in slice 0, or kNowhere
        int k[kVecs];             // its first contraction index in the slice
    };
    __device__ static void lane_offsets(Lane& l, int ld, int row0, int rows) {
#pragma unroll
        for (int q = 0; q < kVecs; ++q) {
            const int v = threadIdx.x + q * kThreads, line = v / kVecLine, e = 8 * (v % kVecLine);
            const int row = KC ? row0 + line : row0 + e;
            l.k[q] = !KC ? line : STRIP ? 16 * (e / 16) + e % 16 / 2 : e;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const bool ok = KC ? row < rows : row + 4 * h < rows;
                l.off[q][h] = ok ? 4u * (unsigned)(KC ? row * ld + l.k[q] + kSecond * h : line * ld + row + 4 * h) : kNowhere;
            }
        }
    }
    // slice at k0 (uniform byte offset `first`), of which klen contraction indices exist
    __device__ static void load(f4 (&r)[kVecs][2], const Lane& l, rsrc_t rs, unsigned first, int klen) {
#pragma unroll
        for (int q = 0; q < kVecs; ++q)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const bool in = l.k[q] + (KC ? kSecond * h : 0) < klen;
                r[q][h] = __builtin_bit_cast(f4, buf_load(rs, in ? l.off[q][h] : kNowhere, first));
            }
    }
    __device__ static uint8_t* place(uint8_t* lds, int q) {
        const int v = threadIdx.x + q * kThreads, line = v / kVecLine, e = v % kVecLine;
        if (KC) return lds + line * kLine + ((e ^ ((line >> 2) & 3)) << 4);
        const int piece = e / 4;   // 64-byte pieces of 32 rows
        const int key = ROWS == 128 ? line & 3 : (line >> 1) & 1;
        return lds + line * kLine + ((piece ^ key) << 6) + (e % 4) * 16;
    }
    template <bool HUGE_VALUES>
    __device__ static void store(uint8_t* lds, const f4 (&r)[kVecs][2], float& top) {
#pragma unroll
        for (int q = 0; q < kVecs; ++q) {
            const Split8 s = HUGE_VALUES ? split8(r[q][0], r[q][1]) : split8_finite(r[q][0], r[q][1], top);
            uint8_t* d = place(lds, q);
            *(u4*)d = s.hi;
            *(u4*)(d + kTerm) = s.mid;
            *(u4*)(d + 2 * kTerm) = s.lo;
        }
    }
    // rows r0 .. r0 + 31 (a multiple of 32), k-step s: lane holds its half's eight indices of 16 s .. 16 s + 15, of row lane % 32
    __device__ static void frag(SplitFrag& f, const uint8_t* lds, int r0, int s, int lane) {
        if constexpr (KC) {
            const int row = r0 + lane % 32, slot = 2 * s + lane / 32;
            const uint8_t* p = lds + row * kLine + ((slot ^ ((row >> 2) & 3)) << 4);
            f.hi = __builtin_bit_cast(bf16x8, *(const u4*)p);
            f.mid = __builtin_bit_cast(bf16x8, *(const u4*)(p + kTerm));
            f.lo = __builtin_bit_cast(bf16x8, *(const u4*)(p + 2 * kTerm));
        } else {
            typedef s4v __attribute__((address_space(3))) * lds_s4_ptr;
            const int blk = lane / 16, j = lane % 16;
            const int line = 16 * s + (STRIP ? 4 : 8) * (blk / 2) + j / 4;
            const int key = ROWS == 128 ? line & 3 : (line >> 1) & 1;   // the same kSecond lines on
            const uint8_t* p = lds + line * kLine + (((r0 / 32) ^ key) << 6) + (16 * (blk % 2) + 4 * (j % 4)) * 2;
            auto term = [&](int t) {
                const s4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(p + t * kTerm));
                const s4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(p + t * kTerm + kSecond * kLine));
                return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            };
            f.hi = term(0);
            f.mid = term(1);
            f.lo = term(2);
        }
    }
};

template <int BM, int BN, int DEPTH, bool STRIP>
__global__ __launch_bounds__(kThreads, 2) void gemm_split_kernel(GemmSDev p) {
    using TA = STile<BM, true, STRIP>;
    using TB = STile<BN, false, STRIP>;
    constexpr int WM = BM / 2, WN = BN / 2, TM = WM / 32, TN = WN / 32;   // 2 x 2 wavefronts
    constexpr int kSlice = TA::kBytes + TB::kBytes;
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * kSlice];
    auto lds_a = [&](int buf) { return lds + buf * kSlice; };
    auto lds_b = [&](int buf) { return lds + buf * kSlice + TA::kBytes; };

    // hardware deals workgroup b to XCD b % 8: each XCD gets a contiguous range of tiles
    const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
    const int tile = xcd * p.chunk + slot;
    if (slot >= p.chunk || tile >= p.total_tiles) return;
    const int per_split = p.tiles_m * p.tiles_n, per_group = per_split * p.splits;
    const int group = tile / per_group;
    const int split = (tile % per_group) / per_split;
    const int tm = (tile % per_split) / p.tiles_n, tn = tile % p.tiles_n;
    const int m0 = tm * BM, n0 = tn * BN;
    const int k_lo = split * p.k_chunk, k_hi = min(p.K, k_lo + p.k_chunk);
    const rsrc_t ra_rs = make_rsrc(p.a + (int64_t)group * p.sa, p.a_bytes);
    const rsrc_t rb_rs = make_rsrc(p.b + (int64_t)group * p.sb, p.b_bytes);

    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int lane32 = lane % 32, half = lane / 32;
    const int wm0 = (wave / 2) * WM, wn0 = (wave % 2) * WN;

    typename TA::Lane la;
    typename TB::Lane lb;
    TA::lane_offsets(la, p.lda, m0, p.M);
    TB::lane_offsets(lb, p.ldb, n0, p.N);
    const unsigned step_a = 4u * kBK, step_b = 4u * kBK * (unsigned)p.ldb;
    const unsigned first_a = 4u * (unsigned)k_lo;
    const unsigned first_b = 4u * (unsigned)k_lo * (unsigned)p.ldb;
    const int nk = (k_hi - k_lo + kBK - 1) / kBK, nkd = (nk + DEPTH - 1) / DEPTH * DEPTH;
    f4 ra[DEPTH][TA::kVecs][2], rb[DEPTH][TB::kVecs][2];
    auto load = [&](int set, int sl) {   // slices past the range are zeros (their uniform offset stays inside the operand)
        const int klen = k_hi - k_lo - sl * kBK;
        const unsigned in = (unsigned)min(sl, nk - 1);
        TA::load(ra[set], la, ra_rs, first_a + in * step_a, klen);
        TB::load(rb[set], lb, rb_rs, first_b + in * step_b, klen);
    };
    float top = 0.0f;
    auto store = [&](int set, int buf) {
        top = 0.0f;
        TA::template store<false>(lds_a(buf), ra[set], top);
        TB::template store<false>(lds_b(buf), rb[set], top);
    };
    // a slice with a value that needs the separate path once more, to the same places.  (From memory: a second use of the
    // register sets behind a branch would keep the compiler from holding them in registers.)
    auto mend = [&](int buf, int sl) {
        if (__builtin_expect(top >= kRoundsToInf, 0)) {
            const int klen = k_hi - k_lo - sl * kBK;
            const unsigned in = (unsigned)min(sl, nk - 1);
            f4 xa[TA::kVecs][2], xb[TB::kVecs][2];
            TA::load(xa, la, ra_rs, first_a + in * step_a, klen);
            TB::load(xb, lb, rb_rs, first_b + in * step_b, klen);
            TA::template store<true>(lds_a(buf), xa, top);
            TB::template store<true>(lds_b(buf), xb, top);
        }
    };

    f16v acc[TN][TM], low[TN][TM];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[j][i][r] = low[j][i][r] = 0.0f;
    SplitFrag fa[2][TM], fb[2][TN];
    auto frags = [&](int buf, int s) {
#pragma unroll
        for (int i = 0; i < TM; ++i) TA::frag(fa[s][i], lds_a(buf), wm0 + 32 * i, s, lane);
#pragma unroll
        for (int j = 0; j < TN; ++j) TB::frag(fb[s][j], lds_b(buf), wn0 + 32 * j, s, lane);
    };
    auto products = [&](int s) {
#pragma unroll
        for (int j = 0; j < TN; ++j) mfma_split(acc[j], low[j], fa[s], fb[s][j]);
    };
    // Slice t feeds the matrix cores from LDS, slices t + 1 .. t + DEPTH - 1 wait in registers or are on their way; slice
    // t + 1 is split into the other buffer between the two halves of slice t, and slice t + DEPTH is requested into the
    // registers that slice t left.
#pragma unroll
    for (int j = 0; j < DEPTH; ++j) load(j, j);
    store(0, 0);
    mend(0, 0);
    __syncthreads();
    for (int kt = 0; kt < nkd; kt += DEPTH) {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            load(u, kt + u + DEPTH);
            frags(u & 1, 0);
            products(0);
            store((u + 1) % DEPTH, (u + 1) & 1);
            frags(u & 1, 1);
            products(1);
            mend((u + 1) & 1, kt + u + 1);
            __syncthreads();
        }
    }

    // register r of a lane holds C[row][col] with col = lane % 32, row = 8 (r / 4) + 4 (lane / 32) + r % 4 of its block
    const bool raw = p.splits > 1;
    float* C = raw ? p.partial + ((int64_t)split * p.groups + group) * p.M * p.N : p.c + (int64_t)group * p.sc;
    const int ldc = raw ? p.N : p.ldc;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = n0 + wn0 + 32 * j + lane32;
            if (col >= p.N) continue;
            float bias = 0.0f;
            if (!raw) bias = p.bias[(int64_t)group * p.sbias + col];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = m0 + wm0 + 32 * i + 8 * (r / 4) + 4 * half + (r % 4);
                if (row >= p.M) continue;
                float v = split_sum(acc[j][i][r], low[j][i][r]);
                if (!raw) v = fmaxf(v + bias, 0.0f);
                C[(int64_t)row * ldc + col] = v;
            }
        }
    }
}

bool aligned16(const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; }

template <int BM, int BN, int DEPTH>
hipError_t gemm_launch(const GemmArgs& g, hipStream_t s) {
    if (!g.a || !g.b || !g.c || !g.bias || g.groups < 1 || g.M < 1 || g.N < 1 || g.K < 1) return hipErrorInvalidValue;
    if (!aligned16(g.a) || !aligned16(g.b) || g.lda % 4 || g.ldb % 4 || g.sa % 4 || g.sb % 4) return hipErrorInvalidValue;
    if (g.K % 4 || g.N % 4) return hipErrorInvalidValue;
    if (g.lda < g.K || g.ldb < g.N || g.ldc < g.N) return hipErrorInvalidValue;
    GemmSDev p = {};
    p.a = (const float*)g.a; p.b = (const float*)g.b; p.c = (float*)g.c;
    p.bias = g.bias;
    p.sa = g.sa; p.sb = g.sb; p.sc = g.sc; p.sbias = g.sbias;
    p.M = g.M; p.N = g.N; p.K = g.K; p.lda = g.lda; p.ldb = g.ldb; p.ldc = g.ldc;
    const int64_t a_elems = (int64_t)(g.M - 1) * g.lda + g.K;
    const int64_t b_elems = (int64_t)(g.K - 1) * g.ldb + g.N;
    if (!gemm_split_fits(a_elems, b_elems)) return hipErrorInvalidValue;
    p.a_bytes = (unsigned)(4 * a_elems);
    p.b_bytes = (unsigned)(4 * b_elems);
    p.tiles_m = (g.M + BM - 1) / BM;
    p.tiles_n = (g.N + BN - 1) / BN;
    p.groups = g.groups;
    p.splits = 1;
    p.k_chunk = g.K;
    if (g.splits > 1) {
        if (!g.partial) return hipErrorInvalidValue;
        p.k_chunk = g.k_chunk ? g.k_chunk : (int)round_up((g.K + g.splits - 1) / g.splits, kBK);
        if (p.k_chunk % kBK) return hipErrorInvalidValue;
        p.splits = (g.K + p.k_chunk - 1) / p.k_chunk;   // never an empty split
        p.partial = g.partial;
    }
    const int64_t total = (int64_t)g.groups * p.splits * p.tiles_m * p.tiles_n;
    if (total > (1 << 30)) return hipErrorInvalidValue;
    p.total_tiles = (int)total;
    p.chunk = (int)((total + kXcds - 1) / kXcds);
    const unsigned grid = (unsigned)(p.chunk * kXcds);
    if (g.strip_order) gemm_split_kernel<BM, BN, DEPTH, true><<<grid, kThreads, 0, s>>>(p);
    else gemm_split_kernel<BM, BN, DEPTH, false><<<grid, kThreads, 0, s>>>(p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.splits == 1) return e;
    return launch_splitk_finish(p.partial, p.splits, g, s);
}

}  // namespace

// A first layer whose weight gradient goes by column strips has its products in the strips' ranges, few of them, whatever its own plan
// would be; callers that drive the steps one by one form them here.  Where 64 x 128 tiles leave much of a round of two per compute
// unit empty, 64 x 64 ones are faster on short contractions of one row of tiles (the same bits).  us per launch, 64 x 128 / 64 x 64: 45 x
// (64 x 512 x 1556), 180 tiles, 65 / 62; 11 x (48 x 1076 x 1220), 198, 37.6 / 35.5; 13 x (40 x 432 x 1544), 208, 21.3 / 19.4; 64 x (24 x 1264 x
// 756), 640, 107 / 94; but longer 14 x (20 x 1768 x 2428), 196, 55 / 60 and 64 x (64 x 1024 x 3072), 512, 189 / 240, more rows 39 x (72 x 300 x
// 1536), 468, 55 / 59, full rounds 39 x (36 x 1620 x 632), 507 (a step with 4 % more).
hipError_t launch_gemm_split_fwd(const GemmArgs& g, hipStream_t s) {
    const int64_t tiles = (int64_t)g.groups * ((g.M + 63) / 64) * ((g.N + 127) / 128) * (g.splits > 1 ? g.splits : 1);
    if (g.strip_order && g.M <= 64 && g.K <= 2048 && tiles <= 320 * ((tiles + 511) / 512)) return gemm_launch<64, 64, 2>(g, s);
    return gemm_launch<64, 128, 4>(g, s);
}

}  // namespace ols
