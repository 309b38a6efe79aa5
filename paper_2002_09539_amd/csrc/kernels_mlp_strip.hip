// Weight gradient of the fp32 MLPs' first hidden layer by column strips, with the fused update, and -- from the very registers that
// hold the new weights -- the forward product of the NEXT step:
//
//   dW = X_t^T dZ;   W' = update(W, dW);   H_{t+1} = relu(X_{t+1} W' + b')
//
// (gradient and local step of Section 2, arXiv 2002.09539; the data are resident and the layer's input needs no earlier layer, so
// ols_run_steps knows X_{t+1}.)  The next forward GEMM would read from memory what this launch has just written, and wait for it.
//
// A workgroup owns 128 columns of a worker and walks down the weight rows, 64 at a time; eight wavefronts own a 32 x 32 block each.
// All products are split ones (split_bf16.h).  The blocks' accumulator registers are updated where they are -- the state is read
// and written one element per lane, two whole 128-byte lines per access -- and go to LDS as ready fragments; wavefront (wr, wc) then
// adds its half of the samples over all 64 rows.  One range of rows per strip finishes the product itself (in the delta's place,
// which nobody else reads); where strips alone do not fill the chip, several ranges leave raw sums and a second pass adds them.
// Without a next step (the last of a call, and all steps of callers that drive them one by one) the same kernel leaves that part
// out, and the forward GEMM of kernels_gemm_split.hip adds the same products in the same order: the same bits either way.
//
// What bounds it: the state, 16 bytes per weight with momentum, walked down in strips: a probe that only streams it in this order
// takes 579 us for 64 x (3072 x 1024) and 80 for 16 x (3072 x 512) (whole tiles side by side 537 and 72; strips of 64 columns 640 and
// 81).  Us per launch, batch 64 and 128: 580 - 640 and 118 - 124 (up to 147 where the clock is still rising), where the weight gradient
// alone took 582 - 602 and 100 - 105 and the forward GEMM 187 and 59 + 6; without the next product 590 - 627 and 102 - 105.  Counters, with
// the product: matrix pipes busy 27 % and 22 - 27 %, 3.44 GB and 0.51 GB moved (3.25 and 0.46 of state and operands).  At batch 128 the
// products are next: the launch takes 103 us with no state at all, vector ALU (splitting, update), LDS and matrix work in phases that
// eight wavefronts in step do not overlap.  Not kept: two elements per access, which costs the exchange of two lanes and touches four
// rows (654 and 144 us); fp32 matrix products for the gradient (631 and 140); at batch 128 the delta split anew for every tile instead of
// by halves (134), at batch 64 by halves as well (601).  Two rounds: 64 x (3072-1024-10, 64) tau 8 12900 -> 10190, 16 x (3072-512-10, 128)
// tau 2 644 -> 567; 40 random MLPs with one hidden layer that take it 1.15 times as fast in the geometric mean, one 2 % slower (20 x
// (1772-672-7, 20) tau 1, 285 and 290 us).
//
// Accuracy: six of the nine bf16 products of every fp32 one, for operands of at least 2^-109 (below, up to 2^-133 of an operand is
// missing; split_bf16.h).  From the same operands, relative 2-norm against 64 bits, over 42 layers (3 - 64 workers, 520 - 3072 x 84 - 2044,
// batch 16 - 128): gradients 2.7e-8 - 4.7e-8, 0.34 - 0.53 times the error of the fp32 matrix cores' 128 x 128 tiles, products 1.0e-7 -
// 3.4e-7, 0.30 - 0.47 times that of their 64 x 64 tiles.
#include "gemm_f32_tile.h"
#include "head_dw_body.h"
#include "mlp_strip_plan.h"
#include "ols_internal.h"
#include "split_bf16.h"

namespace ols {

namespace {

constexpr int kXcds = 8;
constexpr int kThreads = 512;                // eight wavefronts: 2 halves x 4 of 32 columns
constexpr int kRows = kStripRows, kCols = kStripCols;
constexpr int kLine = 3 * 2 * kRows;         // bytes of a sample's rows of a tile in three bf16 terms
constexpr int kWxBytes = 8 * 6 * 1024;       // the wavefronts' new weights as fragments of the products
constexpr int kGxBytes = 8 * 4 * 1024;       // half sums of the gradient on their way to the wavefront that owns their rows
constexpr unsigned kNowhere = kStripNowhere;

struct StripDev {
    const float* xa;     // batch of the step, [B][M] per worker
    const float* dz;     // its delta at the first hidden layer, [B][N]
    const float* xn;     // batch of the next step
    float* out;          // one range: relu(xn W + b), [B][N] per worker; else raw sums, [range][worker][B][N]
    float* g;            // without the update: gradients, sg between workers; weights at upd_w_off, bias at upd_b_off
    int64_t sxa, sdz, sxn, sout, sg;
    FusedUpdate upd;
    int64_t upd_w_off, upd_b_off;
    int M, N, B, groups;
    int strips, ranges, tiles_m, tiles_per_range, total, chunk;
    HeadDwDev guest;
};

template <bool STREAM>
__device__ __forceinline__ float state_load(rsrc_t r, unsigned off) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, STREAM ? 2 : 0));
}
template <bool STREAM>
__device__ __forceinline__ void state_store(float v, rsrc_t r, unsigned off) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)off, 0, STREAM ? 2 : 0);
}

__device__ __forceinline__ void take_terms(SplitFrag& f, const Split8& v) {
    f.hi = __builtin_bit_cast(bf16x8, v.hi);
    f.mid = __builtin_bit_cast(bf16x8, v.mid);
    f.lo = __builtin_bit_cast(bf16x8, v.lo);
}

// NB: blocks of 32 samples.  With 128 samples the terms of a strip's delta are too many for every wavefront's registers: the
// contraction then goes by halves of the samples.
template <int NB>
constexpr bool strip_halves() { return NB > 2; }

// LDS.  By halves the fragments of the new weights take the place of the batch's tile, which the contraction has read by then.
// Before the first tile the strip's delta lies there.
template <int NB, bool FWD>
struct StripLds {
    static constexpr bool kHalves = strip_halves<NB>();
    static constexpr int kTile = NB * 32 * kLine, kDs = NB * 32 * kCols * 4;
    static constexpr int kXs = FWD && kHalves && kWxBytes > kTile ? kWxBytes : kTile;
    static constexpr int kXn = kXs, kWx = kHalves ? 0 : kXn + kTile, kGx = kXn + (FWD ? kTile : 0);   // offsets
    static constexpr int kMost = kHalves ? kGx + kGxBytes : FWD ? kWx + kWxBytes : kXs;
    static constexpr int kBytes = kMost > kDs ? kMost : kDs;
    static_assert(kBytes <= 160 * 1024, "LDS of a compute unit");
};

template <int NB, bool FWD, bool UPD, bool PULL, bool MOM, bool STREAM>
__global__ __launch_bounds__(kThreads, 2) void strip_kernel(StripDev p) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    using Lds = StripLds<NB, FWD>;
    constexpr int kBatch = NB * 32, HB = NB / 2;
    float* ds = (float*)lds;                        // at the start: [kBatch][kCols] the strip's delta
    uint8_t* xs = lds;                              // [kBatch][kLine] the batch's tile, three bf16 terms
    uint8_t* wx = lds + Lds::kWx;
    uint8_t* xn = lds + Lds::kXn;                   // the next batch's
    uint8_t* gx = lds + Lds::kGx;
    float* bs = (float*)lds;                        // at the end: the strip's bias

    int bid = blockIdx.x;
    if (bid < p.guest.blocks) {
        if (threadIdx.x < kHeadDwThreads) head_dw_guest<Lds::kBytes / 4>(p.guest, ds, bid);
        return;
    }
    bid -= p.guest.blocks;
    const int xcd = bid % kXcds, slot = bid / kXcds, unit = xcd * p.chunk + slot;
    if (slot >= p.chunk || unit >= p.total) return;
    const int strip = unit % p.strips, range = (unit / p.strips) % p.ranges, group = unit / (p.strips * p.ranges);
    const int n0 = strip * kCols, M = p.M, N = p.N;
    const int tile0 = range * p.tiles_per_range, tile1 = min(p.tiles_m, tile0 + p.tiles_per_range);

    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, lane32 = lane % 32, half = lane / 32;
    const int wr = wave / 4, wc = wave % 4;
    const int col = n0 + 32 * wc + lane32;
    const FusedUpdate& u = p.upd;
    const unsigned n4 = 4u * (unsigned)N, m4 = 4u * (unsigned)M;
    const unsigned w_bytes = (unsigned)M * n4, x_bytes = (unsigned)p.B * m4;

    const int64_t w_at = (int64_t)group * u.ld + p.upd_w_off;
    const rsrc_t w_rs = make_rsrc(UPD ? u.x_in + w_at : nullptr, UPD ? w_bytes : 0u);
    const rsrc_t wo_rs = make_rsrc(UPD ? u.x_out + w_at : p.g + (int64_t)group * p.sg + p.upd_w_off, w_bytes);
    const rsrc_t b_rs = make_rsrc(MOM ? u.buf + w_at : nullptr, MOM ? w_bytes : 0u);
    const rsrc_t z_rs = make_rsrc(PULL ? u.z + p.upd_w_off : nullptr, PULL ? w_bytes : 0u);
    const rsrc_t xa_rs = make_rsrc(p.xa + (int64_t)group * p.sxa, x_bytes);
    const rsrc_t xn_rs = make_rsrc(FWD ? p.xn + (int64_t)group * p.sxn : nullptr, FWD ? x_bytes : 0u);

    // weight element r of the lane (accumulator order): row 8 (r / 4) + 4 half + r % 4 of the wavefront's 32, column lane % 32
    const unsigned w_lane = col < N ? strip_offset(4u * (unsigned)col, (unsigned)(32 * wr + 4 * half), n4) : kNowhere;
    auto w_off = [&](int row0, int r) { return strip_offset(w_lane, (unsigned)(row0 + 8 * (r / 4) + r % 4), n4); };
    float sx[16], sb[MOM ? 16 : 1], sz[PULL ? 16 : 1];
    auto state_request = [&](int row0) {
        if constexpr (UPD) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const unsigned o = w_off(row0, r);
                sx[r] = state_load<STREAM>(w_rs, o);
                if (MOM) sb[MOM ? r : 0] = state_load<STREAM>(b_rs, o);
            }
        }
    };

    // Tiles of the two batches: a lane takes eight rows of a sample.  Of this step's batch eight in a row, for the transpose loads;
    // of the next one rows 16 s + 4 h + 0 .. 3 and 16 s + 8 + 4 h + 0 .. 3, the order in which the accumulators of lane half h hold
    // the new weights, for 16-byte fragments.
    constexpr int kVecs = kBatch * 8 / kThreads;
    f4 xt[kVecs][2], xr[FWD ? kVecs : 1][2];
    const int x_line = threadIdx.x / 8, x_slot = threadIdx.x % 8;
    auto batch_request = [&](int row0) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = row0 + 8 * x_slot + 4 * h;
            const unsigned o = k < M ? strip_offset(4u * (unsigned)k, (unsigned)x_line, m4) : kNowhere;
#pragma unroll
            for (int t = 0; t < kVecs; ++t) xt[t][h] = __builtin_bit_cast(f4, buf_load(xa_rs, strip_offset(o, (unsigned)(kThreads / 8 * t), m4), 0));
        }
    };
    auto next_request = [&](int row0) {
        if constexpr (FWD) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int k = row0 + 16 * (x_slot / 2) + 4 * (x_slot % 2) + 8 * h;
                const unsigned o = k < M ? strip_offset(4u * (unsigned)k, (unsigned)x_line, m4) : kNowhere;
#pragma unroll
                for (int t = 0; t < kVecs; ++t) xr[t][h] = __builtin_bit_cast(f4, buf_load(xn_rs, strip_offset(o, (unsigned)(kThreads / 8 * t), m4), 0));
            }
        }
    };
    auto batch_store = [&]() {
        auto put = [&](uint8_t* d, const Split8& v) {
            *(u4*)d = v.hi;
            *(u4*)(d + 2 * kRows) = v.mid;
            *(u4*)(d + 4 * kRows) = v.lo;
        };
        auto place = [&](int t) {   // 64-byte pieces trade places by line / 2
            const int line = x_line + kThreads / 8 * t;
            return xs + line * kLine + (((x_slot / 4) ^ (line / 2 % 2)) << 6) + 16 * (x_slot % 4);
        };
        auto place_next = [&](int t) {
            const int line = x_line + kThreads / 8 * t;
            return xn + line * kLine + 16 * (x_slot ^ (line / 2 % 8));
        };
        float top = 0.0f;
#pragma unroll
        for (int t = 0; t < kVecs; ++t) {
            put(place(t), split8_finite(xt[t][0], xt[t][1], top));
            if (FWD) put(place_next(t), split8_finite(xr[FWD ? t : 0][0], xr[FWD ? t : 0][1], top));
        }
        if (__builtin_expect(top >= kRoundsToInf, 0)) {
#pragma unroll
            for (int t = 0; t < kVecs; ++t) {
                put(place(t), split8(xt[t][0], xt[t][1]));
                if (FWD) put(place_next(t), split8(xr[FWD ? t : 0][0], xr[FWD ? t : 0][1]));
            }
        }
    };

    f16v acc[HB], low[HB];
#pragma unroll
    for (int i = 0; i < HB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = low[i][r] = 0.0f;

    {
        constexpr int kVecLine = kCols / 4, kDv = kBatch * kVecLine / kThreads;
        const rsrc_t dz_rs = make_rsrc(p.dz + (int64_t)group * p.sdz, (unsigned)p.B * n4);
        const int line = threadIdx.x / kVecLine, c4 = 4 * (threadIdx.x % kVecLine);
        const unsigned o = n0 + c4 < N ? strip_offset(4u * (unsigned)(n0 + c4), (unsigned)line, n4) : kNowhere;
        f4 dv[kDv];
#pragma unroll
        for (int t = 0; t < kDv; ++t) dv[t] = __builtin_bit_cast(f4, buf_load(dz_rs, strip_offset(o, (unsigned)(kThreads / kVecLine * t), n4), 0));
        batch_request(tile0 * kRows);
        next_request(tile0 * kRows);
#pragma unroll
        for (int t = 0; t < kDv; ++t) {
            const int row = line + kThreads / kVecLine * t;
            *(f4*)(ds + row * kCols + c4) = dv[t];
        }
    }
    // Fragments of the contraction over the samples.  The wavefront's part of the delta stays in registers and is split once: all
    // samples, or (by halves) samples 16 NB wr .., with which it then forms the other half's rows as well.
    constexpr bool kHalves = Lds::kHalves;
    constexpr int S = kHalves ? NB : 2 * NB;
    constexpr bool kLate = PULL && kHalves;   // the anchor's registers are not there for requests ahead
    const int s_first = kHalves ? NB * wr : 0;
    SplitFrag dfr[S];
    __syncthreads();
#pragma unroll
    for (int s = 0; s < S; ++s) {   // samples 16 (s_first + s) + 8 half + 0 .. 7
        const float* d = ds + (16 * (s_first + s) + 8 * half) * kCols + 32 * wc + lane32;
        take_terms(dfr[s], split8(f4{d[0], d[kCols], d[2 * kCols], d[3 * kCols]}, f4{d[4 * kCols], d[5 * kCols], d[6 * kCols], d[7 * kCols]}));
    }
    // the bias' gradient: column sums of the delta in sample order
    const bool bias_lane = range == 0 && (int)threadIdx.x < kCols && n0 + (int)threadIdx.x < N;
    float bias_sum = 0.0f;
    if (bias_lane) {
#pragma unroll 16
        for (int b = 0; b < kBatch; ++b) bias_sum += ds[b * kCols + threadIdx.x];   // (zeros past the batch)
    }
    auto batch_frag = [&](SplitFrag& f, int rows32, int s) {
        typedef s4v __attribute__((address_space(3))) * lds_s4_ptr;
        const int blk = lane / 16, j = lane % 16;
        const int line = 16 * (s_first + s) + 8 * (blk / 2) + j / 4;
        const uint8_t* q = xs + line * kLine + ((rows32 ^ (line / 2 % 2)) << 6) + (16 * (blk % 2) + 4 * (j % 4)) * 2;
        auto term = [&](int t) {   // (four lines on: the same place in the line)
            const s4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(q + t * 2 * kRows));
            const s4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(q + t * 2 * kRows + 4 * kLine));
            return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        };
        f.hi = term(0);
        f.mid = term(1);
        f.lo = term(2);
    };
    __builtin_amdgcn_sched_barrier(0);
    if (!kLate) state_request(tile0 * kRows);
    __builtin_amdgcn_sched_barrier(0);
    for (int tile = tile0; tile < tile1; ++tile) {
        const int row0 = tile * kRows, next0 = min(row0 + kRows, (tile1 - 1) * kRows);
        __syncthreads();   // the previous tile's fragments are read
        batch_store();
        __syncthreads();
        if (kLate) state_request(row0);
        if constexpr (PULL) {
#pragma unroll
            for (int r = 0; r < 16; ++r) sz[PULL ? r : 0] = state_load<false>(z_rs, w_off(row0, r));
            __builtin_amdgcn_sched_barrier(0);
        }
        batch_request(next0);
        if (!kLate) next_request(next0);
        __builtin_amdgcn_sched_barrier(0);
        f16v ga[1], gl[1];
        auto contract = [&](int rows32) {
#pragma unroll
            for (int r = 0; r < 16; ++r) ga[0][r] = gl[0][r] = 0.0f;
            SplitFrag a[2][1];
            batch_frag(a[0][0], rows32, 0);
#pragma unroll
            for (int s = 0; s < S; ++s) {
                if (s + 1 < S) batch_frag(a[(s + 1) & 1][0], rows32, s + 1);
                mfma_split(ga, gl, a[s & 1], dfr[s]);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) ga[0][r] = split_sum(ga[0][r], gl[0][r]);
        };
        if constexpr (kHalves) {   // the other wavefront's rows first: their half sum is on its way while this one's are formed
            uint8_t* give = gx + wave * 4096 + 16 * lane;
            const uint8_t* get = gx + (wave ^ 4) * 4096 + 16 * lane;
            contract(1 - wr);
#pragma unroll
            for (int q = 0; q < 4; ++q) *(f4*)(give + 1024 * q) = f4{ga[0][4 * q], ga[0][4 * q + 1], ga[0][4 * q + 2], ga[0][4 * q + 3]};
            contract(wr);
            __syncthreads();   // (and every fragment of the batch's tile is read)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f4 other = *(const f4*)(get + 1024 * q);
#pragma unroll
                for (int e = 0; e < 4; ++e) ga[0][4 * q + e] += other[e];
            }
        } else {
            contract(wr);
        }
        // the new weights, in accumulator order, and their terms
        float w[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float g = ga[0][r];
            const unsigned o = w_off(row0, r);
            if constexpr (UPD) {
                float be = MOM ? sb[MOM ? r : 0] : 0.0f;
                w[r] = local_step_elem(g, sx[r], be, PULL ? sz[PULL ? r : 0] : 0.0f, u.gamma, u.mu, u.alpha, MOM, u.nesterov != 0, PULL);
                state_store<STREAM>(w[r], wo_rs, o);
                if (MOM) state_store<STREAM>(be, b_rs, o);
            } else {
                state_store<false>(g, wo_rs, o);
            }
        }
        if constexpr (FWD) {   // rows that the last tile does not have: 0 times a delta, which an infinite one makes a NaN
            const int left = M - row0 - 32 * __builtin_amdgcn_readfirstlane(wr);   // (lane masks in scalar registers: there are no vector ones)
#pragma unroll
            for (int r = 0; r < 16; ++r) {   // rows 8 (r / 4) + 4 half + 0 .. 3 are there together: M is a multiple of four
                const uint64_t there = (left > 8 * (r / 4) ? 0xFFFFFFFFull : 0ull) | (left > 8 * (r / 4) + 4 ? 0xFFFFFFFFull << 32 : 0ull);
                w[r] = __builtin_amdgcn_inverse_ballot_w64(there) ? w[r] : 0.0f;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (FWD) {
            uint8_t* mine = wx + wave * 6144 + 16 * lane;
            float top = 0.0f;
            auto quad = [&](int r) { return f4{w[r], w[r + 1], w[r + 2], w[r + 3]}; };
            auto put = [&](int s, const Split8& v) {
                *(u4*)(mine + (3 * s) * 1024) = v.hi;
                *(u4*)(mine + (3 * s + 1) * 1024) = v.mid;
                *(u4*)(mine + (3 * s + 2) * 1024) = v.lo;
            };
#pragma unroll
            for (int s = 0; s < 2; ++s) put(s, split8_finite(quad(8 * s), quad(8 * s + 4), top));
            if (__builtin_expect(top >= kRoundsToInf, 0)) {
#pragma unroll
                for (int s = 0; s < 2; ++s) put(s, split8(quad(8 * s), quad(8 * s + 4)));
            }
            __builtin_amdgcn_sched_barrier(0);
            if (kLate) next_request(next0);
            __builtin_amdgcn_sched_barrier(0);
            if (!kLate) state_request(next0);   // (until the next tile's update)
            __syncthreads();
            // half of the samples over all 64 rows
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const uint8_t* w8 = wx + (s / 2 * 4 + wc) * 6144 + 16 * lane + s % 2 * 3072;
                SplitFrag a[HB], b;
                b.hi = *(const bf16x8*)w8;
                b.mid = *(const bf16x8*)(w8 + 1024);
                b.lo = *(const bf16x8*)(w8 + 2048);
                const int line = 32 * HB * wr + lane32;
#pragma unroll
                for (int i = 0; i < HB; ++i) {
                    const uint8_t* f = xn + (line + 32 * i) * kLine + 16 * ((2 * s + half) ^ (line / 2 % 8));   // (32 lines on: the same place)
                    a[i].hi = *(const bf16x8*)f;
                    a[i].mid = *(const bf16x8*)(f + 2 * kRows);
                    a[i].lo = *(const bf16x8*)(f + 4 * kRows);
                }
                mfma_split(acc, low, a, b);
            }
        } else if (!kLate) {
            state_request(next0);
        }
    }

    __syncthreads();   // the last tile's fragments are read
    if (bias_lane) {   // the first range's workgroup updates the bias on the spot
        const int64_t at = p.upd_b_off + n0 + threadIdx.x, idx = (int64_t)group * u.ld + at;
        if constexpr (UPD) {
            float be = MOM ? u.buf[idx] : 0.0f;
            const float v = local_step_elem(bias_sum, u.x_in[idx], be, PULL ? u.z[at] : 0.0f, u.gamma, u.mu, u.alpha, MOM, u.nesterov != 0, PULL);
            if (MOM) u.buf[idx] = be;
            u.x_out[idx] = v;
            if (FWD) bs[threadIdx.x] = v;
        } else {
            p.g[(int64_t)group * p.sg + at] = bias_sum;
        }
    }
    if constexpr (FWD) {
        __syncthreads();
        const bool raw = p.ranges > 1;
        const rsrc_t out_rs = make_rsrc(p.out + (raw ? ((int64_t)range * p.groups + group) * p.B * N : (int64_t)group * p.sout), (unsigned)p.B * n4);
        const float bias = raw || col >= N ? 0.0f : bs[32 * wc + lane32];
        const unsigned o = col < N ? strip_offset(4u * (unsigned)col, (unsigned)(32 * HB * wr + 4 * half), n4) : kNowhere;
#pragma unroll
        for (int i = 0; i < HB; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float v = split_sum(acc[i][r], low[i][r]);
                if (!raw) v = fmaxf(v + bias, 0.0f);
                state_store<false>(v, out_rs, strip_offset(o, (unsigned)(32 * i + 8 * (r / 4) + r % 4), n4));   // samples past the batch are dropped
            }
    }
}

bool aligned16(const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; }

template <int NB, bool FWD, bool UPD, bool PULL, bool MOM, bool STREAM>
hipError_t strip_launch(const StripDev& p, hipStream_t s) {
    constexpr size_t bytes = StripLds<NB, FWD>::kBytes;
    hipError_t e = ensure_dynamic_lds((const void*)strip_kernel<NB, FWD, UPD, PULL, MOM, STREAM>, bytes);
    if (e != hipSuccess) return e;
    strip_kernel<NB, FWD, UPD, PULL, MOM, STREAM><<<(unsigned)(p.guest.blocks + p.chunk * kXcds), kThreads, bytes, s>>>(p);
    return hipGetLastError();
}

template <int NB, bool FWD>
hipError_t strip_dispatch(const StripDev& p, hipStream_t s) {
    // A strip's rows are four lines: non-temporal only where a row is whole lines.  (Where it is halves, which the tiles of the other
    // weight gradients stream, two rounds, us, three states in turn, non-temporal / plain: 12 x (3072-656-10, 64) tau 4 925 / 855, 16 x
    // (3072-528-10, 128) 681 / 668, 50 x (1800-624-10, 64) tau 8 3647 / 3565, 64 x (756-1264-9, 24) tau 4 2159 / 2085.)
    const bool stream = !p.upd.cached && p.N % 32 == 0 && p.upd_w_off % 32 == 0;
    const bool mom = p.upd.mu != 0.0f, pull = p.upd.pull != 0;
#define OLS_STRIP(P, Mo) (stream ? strip_launch<NB, FWD, true, P, Mo, true>(p, s) : strip_launch<NB, FWD, true, P, Mo, false>(p, s))
    if (pull) return mom ? OLS_STRIP(true, true) : OLS_STRIP(true, false);
    return mom ? OLS_STRIP(false, true) : OLS_STRIP(false, false);
#undef OLS_STRIP
}

}  // namespace

hipError_t launch_mlp_strip(const GemmArgs& g, const MlpStripNext* next, hipStream_t s) {
    if (!g.a || !g.b || !g.c || !g.colsum || g.groups < 1 || g.K < 1 || g.K > 128 || g.M < 4 || g.M % 4 || g.N < 4 || g.N % 4) return hipErrorInvalidValue;
    if (!aligned16(g.a) || g.sa % 4 || !aligned16(g.b) || g.sb % 4 || g.lda != g.M || g.ldb != g.N || g.ldc != g.N) return hipErrorInvalidValue;
    if (!mlp_strip_offsets_fit(g.K, g.N, g.M)) return hipErrorInvalidValue;
    if (next && (!g.upd.enabled || !next->x || !aligned16(next->x) || !next->out || !next->bias || next->ranges < 1 || (next->ranges > 1 && !next->partial)))
        return hipErrorInvalidValue;
    StripDev p = {};
    p.M = g.M; p.N = g.N; p.B = g.K; p.groups = g.groups;
    p.xa = (const float*)g.a; p.sxa = g.sa;
    p.dz = (const float*)g.b; p.sdz = g.sb;
    if (g.upd.enabled) {
        if (!g.upd.x_in || !g.upd.x_out || (g.upd.mu != 0.0f && !g.upd.buf) || (g.upd.pull && !g.upd.z) || g.upd.shadow) return hipErrorInvalidValue;
        p.upd = g.upd;
        p.upd_w_off = g.upd_w_off; p.upd_b_off = g.upd_b_off;
    } else {
        p.g = (float*)g.c;
        p.sg = g.sc;
        p.upd_b_off = g.colsum - (float*)g.c;
        if (g.scolsum != g.sc) return hipErrorInvalidValue;
    }
    if (g.guest) {
        hipError_t e = head_dw_prepare(*g.guest, &p.guest);
        if (e != hipSuccess) return e;
    }
    p.strips = (g.N + kCols - 1) / kCols;
    p.tiles_m = (g.M + kRows - 1) / kRows;
    const int ranges = next ? next->ranges : mlp_strip_alone_ranges(g.groups, g.N, g.M, g.splits > 1 ? g.splits : 1, g.upd.enabled != 0);
    p.tiles_per_range = (p.tiles_m + ranges - 1) / ranges;
    p.ranges = (p.tiles_m + p.tiles_per_range - 1) / p.tiles_per_range;
    const bool raw = next && p.ranges > 1;
    if (next) {
        p.xn = next->x; p.sxn = g.sa;
        p.out = raw ? next->partial : next->out;
        p.sout = (int64_t)g.K * g.N;
    }
    const int64_t total = (int64_t)g.groups * p.strips * p.ranges;
    if (total > (1 << 30)) return hipErrorInvalidValue;
    p.total = (int)total;
    p.chunk = (int)((total + kXcds - 1) / kXcds);
    hipError_t e;
    const bool few = g.K <= 64;
    if (!g.upd.enabled) e = few ? strip_launch<2, false, false, false, false, false>(p, s) : strip_launch<4, false, false, false, false, false>(p, s);
    else if (next) e = few ? strip_dispatch<2, true>(p, s) : strip_dispatch<4, true>(p, s);
    else e = few ? strip_dispatch<2, false>(p, s) : strip_dispatch<4, false>(p, s);
    if (e != hipSuccess || !raw) return e;
    GemmArgs f = {};
    f.bias = next->bias; f.sbias = g.upd.ld;
    f.c = next->out; f.sc = p.sout; f.ldc = g.N;
    f.groups = g.groups; f.M = g.K; f.N = g.N;
    return launch_splitk_finish(next->partial, p.ranges, f, s);
}

}  // namespace ols
