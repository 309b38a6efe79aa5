// 3 x 3 convolutions (stride 1, zero padding 1) of the fp32 residual block on the bf16 matrix cores, every fp32 operand
// split exactly into three bf16 terms (split_bf16.h: fp32 accuracy, six bf16 products per fp32 product): forward,
// back-propagated delta and kernel / bias gradient, grouped over the m workers.  Operands, results and layouts are those
// of kernels_conv.hip -- activations [group][P][C] fp32 with P = B H W pixels, kernels [group][9][C][C] -- whose kernels
// stay for the shapes these do not take (conv3x3_split_fits: channels a multiple of 32, images up to about 60 pixels wide).
//
// What bounds it: 154.6 GFLOP per launch at the benchmark shape (16 workers x 128 samples x 32 x 32 x 64 channels) are
// 980 us on the fp32 matrix cores and 6 x 154.6 / 2500 = 371 us on the bf16 ones; the fp32 kernels take 1350 - 1410 us.
//
// FWD / DX: one workgroup per 128 consecutive pixels x 64 output channels.  The pixels a tile reads -- its own and the
// neighbours of nine taps -- are copied to LDS once per 32-channel chunk, split on the way (a strip of rows with hi, mid
// and lo side by side), and the nine taps read their fragments from it: an operand element is split once and used in
// 9 x 64 products.  Rows of the strip follow the VIRTUAL pixel order: one zero column between image rows and one zero
// row between images, v = (n (H + 1) + y + 1) (W + 1) + x + 1, so that a tap is one shift of the row index for every
// pixel and the zeros around an image cost LDS rows, not products (a tile holds image pixels only).
// The kernels are split once per step into the order in which a tap's slice lies in LDS (split_weights_kernel).
//
// Measured at the benchmark shape, us per launch: forward 1350 -> 710 - 790, delta 1410 -> 715 - 760, kernel gradient
// 1415 -> 740 - 780 (with its finish pass); the normalised fp32 block 8.15 -> 5.0 ms per step.  Counters: the matrix pipes
// are busy 68 % (forward) and 72 % (kernel gradient) of the cycles at an engine clock of 1.73 GHz -- the chip lowers its
// clock under this load, so the 371 us of the nominal clock are 510 us here.  On the way: kernel slices double-buffered
// and every tap's fragments requested after its barrier 900 us, three slices and the next fragments requested across the
// barrier 710 us.  The forward epilogue leaves per-tile statistics for a batch normalisation that follows (two passes over
// the 128 rows that the lanes still hold): the normalisation's forward calls 305 -> 195 us, the convolution + 10 us.
// The rule (conv3x3_split_fits): channels in whole 32-channel chunks, strips of at most 320 rows, so that two workgroups share
// a compute unit's LDS (up to 256 rows) or one has it alone, and a halo that the kernel gradient's ring holds.  Images up to
// 61 pixels wide fit unless they are low and wide (1 x 20, 2 x 50) or tiny (1 x 1 .. 2 x 1); everything else keeps the fp32
// kernels.  Output channels are padded to 64: with 32 half of a tile's products are wasted, with 96 a quarter, and the fp32
// kernels waste as many.  Against them, us per two rounds of two steps: 16 workers x 32 samples x 32 x 32 x 32 channels 5348
// and 2492, 4 x 8 x 20 x 20 x 32 899 and 425, 1 x 2 x 3 x 3 x 32 387 and 291; 16 x 16 x 16 x 16 x 96 3337 and 1768, 1 x 8 x 8 x 8 x
// 96 1082 and 572, 16 x 4 x 6 x 6 x 96 normalised 1147 and 850; 1 x 4 x 4 x 4 x 256 1612 and 913; of 240 random shapes of up to
// 60 x 60 pixels none of this route was slower.
#include <algorithm>

#include "fast_div.h"
#include "ols_internal.h"
#include "split_bf16.h"

namespace ols {

namespace {

constexpr int kThreads = kTileThreads;
constexpr int kXcds = 8;
constexpr int kBM = 128;          // pixels per forward / delta tile
constexpr int kBN = 64;           // output-channel tile
constexpr int kKC = 32;           // contraction channels per chunk
constexpr int kRow = 192;         // bytes of a strip (or kernel slice) row: 32 channels x 3 terms x 2 bytes
constexpr int kSlice = kBN * kRow;            // one tap's kernel slice: 64 rows
constexpr int kMaxStripRows = 320;
constexpr int kStagePitch = kBN + 4;          // floats; output staging, 32 rows per wavefront
constexpr int kStageBytes = kBM * kStagePitch * 4;

struct ConvSDev {
    const float* in;
    const uint8_t* w;        // split kernels: [group][chunk][n tile][tap] slices of kSlice bytes
    float* out;
    const float* bias;
    const float* residual;
    const float* mask;
    float* stat_part;        // FWD, optional: [group][tiles_m][3][C] statistics of the tile's rows (count, mean, sum of
                             // squared deviations), which the normalisation that follows merges instead of reading out
    int64_t s_in, s_w, s_out, s_bias, s_res, s_mask;
    int groups, B, H, W, C, P;
    int relu;
    int strip_rows, strip_bytes;
    int tiles_m, tiles_n, total_tiles, chunk;
    FastDiv div_hw, div_w, div_s, div_w1, div_pg, div_tn;   // by H W, W, (H + 1)(W + 1), W + 1, tiles per group, tiles_n
};

__device__ __forceinline__ int xcd_tile(int chunk, int total) {
    const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
    const int tile = xcd * chunk + slot;
    return (slot >= chunk || tile >= total) ? -1 : tile;
}

// Byte address of 16-byte slot `slot` (eight channels) of a strip or slice row, term 0; the other terms lie 64 and 128
// bytes on.  Rows are 192 bytes, so four consecutive rows cover the 64 banks once; the slots of the next four rows are
// exchanged, and the 16 rows of a read phase touch every bank once.
__device__ __forceinline__ int slot_addr(int row, int slot) { return row * kRow + ((slot ^ ((row >> 2) & 3)) << 4); }

// virtual index of image pixel p
__device__ __forceinline__ int virtual_index(const ConvSDev& p, int pix) {
    const int n = (int)fast_div((unsigned)pix, p.div_hw), rem = pix - n * (p.H * p.W);
    const int y = (int)fast_div((unsigned)rem, p.div_w), x = rem - y * p.W;
    return (n * (p.H + 1) + y + 1) * (p.W + 1) + x + 1;
}

// ---------------------------------------------------------------------------------------------
// kernels -> split slices.  Slice (group, chunk, n tile, tap): row n (0 .. 63), 32 contraction channels, three terms.
// FWD: n = output channel, k = input channel; DX: n = input channel, k = output channel.  One lane per row slot.
// ---------------------------------------------------------------------------------------------
struct SplitWeights {
    const float* w[3];       // [group] + s_w: fp32 kernels [9][C][C]
    uint8_t* dst[3];
    int dx[3];
    int64_t s_w, s_dst;
    int C, tiles_n;
};
__global__ __launch_bounds__(256) void split_weights_kernel(SplitWeights p) {
    const int chunks = p.C / kKC;
    const int which = blockIdx.z, group = blockIdx.y;
    const int tap = blockIdx.x % 9, tile = blockIdx.x / 9;          // tile = chunk * tiles_n + n tile
    const int c0 = (tile / p.tiles_n) * kKC, n0 = (tile % p.tiles_n) * kBN;
    if (c0 >= chunks * kKC) return;
    const float* W = p.w[which] + (int64_t)group * p.s_w + (int64_t)tap * p.C * p.C;
    uint8_t* D = p.dst[which] + (int64_t)group * p.s_dst + ((int64_t)tile * 9 + tap) * kSlice;
    // lane -> (row, slot): FWD walks the rows fastest (the output channel is contiguous in memory)
    const int row = threadIdx.x % kBN, slot = threadIdx.x / kBN;
    const int n = n0 + row, k = c0 + 8 * slot;
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int64_t i = p.dx[which] ? (int64_t)n * p.C + k + e : (int64_t)(k + e) * p.C + n;
        x[e] = n < p.C ? W[i] : 0.0f;
    }
    const Split8 s = split8(f4{x[0], x[1], x[2], x[3]}, f4{x[4], x[5], x[6], x[7]});
    uint8_t* d = D + slot_addr(row, slot);
    *(u4*)d = s.hi;
    *(u4*)(d + 64) = s.mid;
    *(u4*)(d + 128) = s.lo;
}

// ---------------------------------------------------------------------------------------------
// forward (MODE 0) and back-propagated delta (MODE 1); NV: strip rows / 64, rounded up
// ---------------------------------------------------------------------------------------------
template <int MODE, int NV>
__global__ __launch_bounds__(kThreads, 2) void conv3x3_split_kernel(ConvSDev p) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    uint8_t* strip = lds;
    auto slice = [&](int buf) { return lds + p.strip_bytes + buf * kSlice; };

    const int tile = xcd_tile(p.chunk, p.total_tiles);
    if (tile < 0) return;
    const int per_group = p.tiles_m * p.tiles_n;
    const int group = (int)fast_div((unsigned)tile, p.div_pg);
    const int in_group = tile - group * per_group;
    const int tm = (int)fast_div((unsigned)in_group, p.div_tn), tn = in_group - tm * p.tiles_n;
    const int m0 = tm * kBM, n0 = tn * kBN;
    const int C = p.C, W1 = p.W + 1;
    const int chunks = C / kKC;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int lane32 = lane % 32, half = lane / 32;

    const unsigned row_bytes = 4u * (unsigned)C;
    const unsigned tensor_bytes = (unsigned)p.P * row_bytes;
    const rsrc_t in_rs = make_rsrc(p.in + (int64_t)group * p.s_in, tensor_bytes);
    const int64_t slices = (int64_t)chunks * p.tiles_n * 9;
    const rsrc_t w_rs = make_rsrc(p.w + (int64_t)group * p.s_w, (unsigned)(slices * kSlice));

    // Strip rows: virtual indices v0 .. v0 + strip_rows - 1.  Lane t owns channels 8 (t % 4) .. of rows t / 4 + 64 i.
    const int v0 = virtual_index(p, m0) - (W1 + 1);
    unsigned strip_off[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int v = v0 + (int)threadIdx.x / 4 + 64 * i;
        const int S = (p.H + 1) * W1;
        const int n = (int)fast_div((unsigned)v, p.div_s), rem = v - n * S;
        const int yy = (int)fast_div((unsigned)rem, p.div_w1), xx = rem - yy * W1;
        const bool img = yy >= 1 && xx >= 1 && n < p.B;
        // zeros around the images: an offset that the range check answers with zeros
        strip_off[i] = img ? (unsigned)((n * p.H + yy - 1) * p.W + xx - 1) * row_bytes + (threadIdx.x % 4) * 32u : 0xFFFFFF00u;
    }
    f4 rs[NV][2];
    auto load_strip = [&](int c0) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const unsigned o = strip_off[i] == 0xFFFFFF00u ? 0xFFFFFF00u : strip_off[i] + 4u * (unsigned)c0;
            rs[i][0] = __builtin_bit_cast(f4, buf_load(in_rs, o, 0u));
            rs[i][1] = __builtin_bit_cast(f4, buf_load(in_rs, o + 16u, 0u));
        }
    };
    auto store_strip = [&]() {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int row = (int)threadIdx.x / 4 + 64 * i;
            if (i >= 2 && row >= p.strip_rows) break;   // (a strip has more than 128 rows)
            const Split8 s = split8(rs[i][0], rs[i][1]);
            uint8_t* d = strip + slot_addr(row, threadIdx.x % 4);
            *(u4*)d = s.hi;
            *(u4*)(d + 64) = s.mid;
            *(u4*)(d + 128) = s.lo;
        }
    };
    constexpr int kWVec = kSlice / (16 * kThreads);   // 3 vectors of a slice per lane
    u4 rw[2][kWVec];
    auto load_w = [&](u4 (&r)[kWVec], int c, int tap) {
        const unsigned first = (unsigned)((c * p.tiles_n + tn) * 9 + tap) * (unsigned)kSlice;
#pragma unroll
        for (int t = 0; t < kWVec; ++t) r[t] = buf_load(w_rs, threadIdx.x * 16u + t * (16u * kThreads), first);
    };
    auto store_w = [&](int buf, const u4 (&r)[kWVec]) {
#pragma unroll
        for (int t = 0; t < kWVec; ++t) *(u4*)(slice(buf) + threadIdx.x * 16 + t * (16 * kThreads)) = r[t];
    };

    // A wavefront owns 32 pixels x 64 channels.  The kernel fragment goes first, so a lane's accumulator quads are four
    // consecutive channels of pixel lane % 32.
    const int own = min(m0 + wave * 32 + lane32, p.P - 1);
    const int own_row = virtual_index(p, own) - v0;
    f16v acc[2], low[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = low[j][r] = 0.0f;
    SplitFrag fa[2], fb[2][2];
    auto load_a = [&](int buf, int row, int s) {
        const uint8_t* a = strip + slot_addr(row, 2 * s + half);
        fa[buf].hi = __builtin_bit_cast(bf16x8, *(const u4*)a);
        fa[buf].mid = __builtin_bit_cast(bf16x8, *(const u4*)(a + 64));
        fa[buf].lo = __builtin_bit_cast(bf16x8, *(const u4*)(a + 128));
    };
    auto load_b = [&](int buf, const uint8_t* w, int s) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint8_t* b = w + slot_addr(32 * j + lane32, 2 * s + half);
            fb[buf][j].hi = __builtin_bit_cast(bf16x8, *(const u4*)b);
            fb[buf][j].mid = __builtin_bit_cast(bf16x8, *(const u4*)(b + 64));
            fb[buf][j].lo = __builtin_bit_cast(bf16x8, *(const u4*)(b + 128));
        }
    };

    // Three kernel slices in LDS: while tap t's feeds the matrix cores, slice t + 1 is in place -- its first fragments are
    // requested ahead of tap t's last products, across the barrier -- and slice t + 2 is being written.
    load_w(rw[0], 0, 0);
    load_w(rw[1], 0, 1);
    load_strip(0);
    for (int c = 0; c < chunks; ++c) {
        // the previous chunk's last barrier has passed: nobody reads the strip or the slices any more
        store_w(0, rw[0]);
        store_w(1, rw[1]);
        load_w(rw[0], c, 2);
        store_strip();
        __syncthreads();
        auto row_of = [&](int tap) { return own_row + (MODE == 0 ? 1 : -1) * ((tap / 3 - 1) * W1 + tap % 3 - 1); };
        load_a(0, row_of(0), 0);
        load_b(0, slice(0), 0);
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            if (tap + 3 < 9) load_w(rw[(tap + 1) % 2], c, tap + 3);
            if (tap == 2 && c + 1 < chunks) load_strip((c + 1) * kKC);
            if (tap == 7 && c + 1 < chunks) {
                load_w(rw[0], c + 1, 0);
                load_w(rw[1], c + 1, 1);
            }
            load_a(1, row_of(tap), 1);
            load_b(1, slice(tap % 3), 1);
            __builtin_amdgcn_sched_barrier(0);
            mfma_split(acc, low, fb[0], fa[0]);
            __builtin_amdgcn_sched_barrier(0);
            if (tap + 1 < 9) {
                load_a(0, row_of(tap + 1), 0);
                load_b(0, slice((tap + 1) % 3), 0);
            }
            if (tap + 2 < 9) store_w((tap + 2) % 3, rw[tap % 2]);
            __builtin_amdgcn_sched_barrier(0);
            mfma_split(acc, low, fb[1], fa[1]);
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
        }
    }

    // Epilogue: the wavefront's 32 rows go through LDS (the strip's place), then 16-byte vectors of whole rows.
    float* stage = (float*)lds + wave * 32 * kStagePitch;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4)
            *(f4*)(stage + lane32 * kStagePitch + 32 * j + 8 * g4 + 4 * half) =
                f4{split_sum(acc[j][4 * g4], low[j][4 * g4]), split_sum(acc[j][4 * g4 + 1], low[j][4 * g4 + 1]),
                   split_sum(acc[j][4 * g4 + 2], low[j][4 * g4 + 2]), split_sum(acc[j][4 * g4 + 3], low[j][4 * g4 + 3])};
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int cq = lane % 16, r0 = lane / 16;                 // channel quad and first row of this lane: rows r0 + 4 t
    const int col = n0 + 4 * cq;
    if (col >= C) return;
    const unsigned first = (unsigned)(m0 + wave * 32 + r0) * row_bytes + 4u * (unsigned)col;
    const rsrc_t out_rs = make_rsrc(p.out + (int64_t)group * p.s_out, tensor_bytes);
    f4 extra[8];
    const bool with_extra = MODE == 0 ? p.residual != nullptr : p.mask != nullptr;
    const float* E = MODE == 0 ? p.residual : p.mask;
    const rsrc_t ex_rs = make_rsrc(with_extra ? E + (int64_t)group * (MODE == 0 ? p.s_res : p.s_mask) : p.in, with_extra ? tensor_bytes : 0u);
#pragma unroll
    for (int t = 0; t < 8; ++t) extra[t] = __builtin_bit_cast(f4, buf_load(ex_rs, first + (unsigned)t * 4u * row_bytes, 0u));
    f4 bias = {0.f, 0.f, 0.f, 0.f};
    if (MODE == 0 && p.bias) {
#pragma unroll
        for (int e = 0; e < 4; ++e) bias[e] = p.bias[(int64_t)group * p.s_bias + col + e];
    }
    f4 v[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        v[t] = *(const f4*)(stage + (r0 + 4 * t) * kStagePitch + 4 * cq);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (MODE == 0) {
                v[t][e] += bias[e];
                if (with_extra) v[t][e] += extra[t][e];
                if (p.relu) v[t][e] = fmaxf(v[t][e], 0.0f);
            } else if (with_extra) {
                v[t][e] = extra[t][e] > 0.0f ? v[t][e] : 0.0f;
            }
        }
        buf_store(__builtin_bit_cast(u4, v[t]), out_rs, first + (unsigned)t * 4u * row_bytes);   // rows past the tensor are dropped
    }
    if constexpr (MODE == 0) {
        // Two passes over the tile's rows, which the lanes still hold, so nothing cancels; a channel quad's sixteen lanes
        // (four per wavefront) are added through LDS in lane order.  (Channels are whole tiles here: nobody has returned.)
        if (p.stat_part) {
            const int rows = min(kBM, p.P - m0);
            const float inv = 1.0f / (float)rows;
            f4* red = (f4*)lds;
            f4 mean = {0.f, 0.f, 0.f, 0.f}, m2 = mean;
            auto add_up = [&](f4 mine) {
                __syncthreads();
                red[threadIdx.x] = mine;
                __syncthreads();
                f4 sum = red[cq];
#pragma unroll
                for (int k = 1; k < 16; ++k) sum = sum + red[16 * k + cq];
                return sum;
            };
            f4 part = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 8; ++t)
                if (wave * 32 + r0 + 4 * t < rows) part = part + v[t];
            part = add_up(part);
#pragma unroll
            for (int e = 0; e < 4; ++e) mean[e] = part[e] * inv;
            part = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 8; ++t)
                if (wave * 32 + r0 + 4 * t < rows) part = part + (v[t] - mean) * (v[t] - mean);
            m2 = add_up(part);
            if (threadIdx.x < 16) {
                float* o = p.stat_part + (((int64_t)group * p.tiles_m + tm) * 3) * C + col;
                *(f4*)o = f4{(float)rows, (float)rows, (float)rows, (float)rows};
                *(f4*)(o + C) = mean;
                *(f4*)(o + 2 * C) = m2;
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// kernel / bias gradient: dw[tap][ci][co] = sum_v in[v + shift(tap)][ci] dout[v][co] over the virtual pixels (where v is no
// image pixel dout counts as zero).  One workgroup per (group, virtual range, 64 x 64 block of input x output channels):
// twelve wavefronts, four per kernel row, 32 x 32 channels x three taps each (48 accumulators per lane), three
// wavefronts per SIMD.  48 pixels per slice: the input rows live in a RING of 256 LDS rows, so that every input row is
// fetched and split once although nine taps read it at nine offsets; the delta's rows alternate between two buffers.
// 64 channels of a row are 128 bytes per term, 384 bytes in all; the 64-byte halves of a term are exchanged by bit 1 of
// the row, so the four rows of a transpose read cover the 64 banks.
// ---------------------------------------------------------------------------------------------
constexpr int kDwThreads = 768, kDwBK = 48, kDwRing = 256, kDwRow = 384;
constexpr int kDwMaxHalo = (kDwRing - 2 * kDwBK) / 2;

struct ConvSDwDev {
    const float* in;
    const float* dout;
    float* partial;          // [splits][groups][9 C C + C]
    int64_t s_in, s_dout;
    int groups, B, H, W, C, V, halo;
    int splits, k_chunk, blocks_n, total_tiles, chunk;
    unsigned tensor_bytes;
    FastDiv div_s, div_w1;
};

// image pixels with a virtual index below v (clamped to the tensor)
__device__ int image_pixels_before(const ConvSDwDev& p, int v) {
    if (v <= 0) return 0;
    if (v >= p.V) return p.B * p.H * p.W;
    const int W1 = p.W + 1, S = (p.H + 1) * W1;
    const int n = (int)fast_div((unsigned)v, p.div_s), rem = v - n * S;
    const int y = (int)fast_div((unsigned)rem, p.div_w1) - 1, x = rem - (y + 1) * W1 - 1;
    return (n * p.H + max(y, 0)) * p.W + (y < 0 ? 0 : max(x, 0));
}
// one element of the kernel gradient over the image pixels of a virtual range
__device__ float pixel_sum(const ConvSDwDev& p, int group, int lo, int hi, int tap, int ci, int co) {
    const float* IN = p.in + (int64_t)group * p.s_in;
    const float* DOUT = p.dout + (int64_t)group * p.s_dout;
    const int W1 = p.W + 1, S = (p.H + 1) * W1, dy = tap / 3 - 1, dx = tap % 3 - 1;
    float sum = 0.0f;
    for (int v = lo; v < hi; ++v) {
        const int n = (int)fast_div((unsigned)v, p.div_s), rem = v - n * S;
        const int y = (int)fast_div((unsigned)rem, p.div_w1) - 1, x = rem - (y + 1) * W1 - 1;
        if (y < 0 || x < 0 || y + dy < 0 || y + dy >= p.H || x + dx < 0 || x + dx >= p.W) continue;
        const int64_t pix = ((int64_t)n * p.H + y) * p.W + x;
        sum = __fmaf_rn(IN[(pix + dy * p.W + dx) * p.C + ci], DOUT[pix * p.C + co], sum);
    }
    return sum;
}

__global__ __launch_bounds__(kDwThreads, 3) void conv3x3_split_dw_kernel(ConvSDwDev p) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    uint8_t* ring = lds;
    auto delta = [&](int buf) { return lds + kDwRing * kDwRow + buf * (kDwBK * kDwRow); };
    const int tile = xcd_tile(p.chunk, p.total_tiles);
    if (tile < 0) return;
    const int nb = p.blocks_n, per_group = p.splits * nb * nb;
    const int group = tile / per_group, rest = tile % per_group;
    const int split = rest / (nb * nb);
    const int ci0 = ((rest / nb) % nb) * 64, co0 = (rest % nb) * 64;
    const int lo = split * p.k_chunk, hi = min(p.V, lo + p.k_chunk);
    const int C = p.C, W1 = p.W + 1, S = (p.H + 1) * W1;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int kh = wave / 4, wi = (wave / 2) % 2, wj = wave % 2;

    // Copying: lanes 0 .. 383 move input rows, 384 .. 767 delta rows; eight channels of one of 48 rows each.
    const bool moves_in = threadIdx.x < kDwThreads / 2;
    const int mt = moves_in ? threadIdx.x : threadIdx.x - kDwThreads / 2;
    const int mrow = mt / 8, mch = (mt % 8) * 8;
    const unsigned row_bytes = 4u * (unsigned)C;
    const int ch = (moves_in ? ci0 : co0) + mch;
    const rsrc_t rs = make_rsrc(moves_in ? p.in + (int64_t)group * p.s_in : p.dout + (int64_t)group * p.s_dout, p.tensor_bytes);
    const int last = moves_in ? 0x7FFFFFFF : hi;   // the delta of other ranges counts as zero
    f4 r0, r1;
    auto load_row = [&](int v) {
        const unsigned vc = v < 0 ? 0u : (unsigned)v;
        const int n = (int)fast_div(vc, p.div_s), rem = (int)vc - n * S;
        const int yy = (int)fast_div((unsigned)rem, p.div_w1), xx = rem - yy * W1;
        const bool img = v >= 0 && v < last && yy >= 1 && xx >= 1 && n < p.B && ch < C;
        const unsigned o = img ? (unsigned)((n * p.H + yy - 1) * p.W + xx - 1) * row_bytes + 4u * (unsigned)ch : 0xFFFFFF00u;
        r0 = __builtin_bit_cast(f4, buf_load(rs, o, 0u));
        r1 = __builtin_bit_cast(f4, buf_load(rs, o + 16u, 0u));
    };
    auto put_row = [&](uint8_t* base, int row) {
        const Split8 s = split8(r0, r1);
        uint8_t* d = base + row * kDwRow + (((mch / 32) ^ ((row >> 1) & 1)) * 64) + (mch % 32) * 2;
        *(u4*)d = s.hi;
        *(u4*)(d + 128) = s.mid;
        *(u4*)(d + 256) = s.lo;
    };
    // the bias gradient is the delta's column sum: eight channels of every 48th row per copying lane
    const bool col_sums = ci0 == 0;
    f4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;

    // fragments (transpose reads): lane's row within a 16-row step, and its column bytes inside the 64-byte half
    const int blk = lane / 16, j = lane % 16;
    const int frow = 8 * (blk / 2) + j / 4, fcol = (16 * (blk % 2) + 4 * (j % 4)) * 2;
    typedef s4v __attribute__((address_space(3))) * lds_s4_ptr;
    auto tr = [](const uint8_t* q) { return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)q); };
    auto frag = [&](const uint8_t* a, const uint8_t* b, int term) {
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(tr(a + 128 * term), tr(b + 128 * term), 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto half_addr = [&](int row, int half) { return row * kDwRow + ((half ^ ((row >> 1) & 1)) * 64) + fcol; };
    f16v acc[3], low[3];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = low[t][r] = 0.0f;

    // ring row of virtual index v: (v - lo + halo) mod 256
    const int nslices = hi > lo ? (hi - lo + kDwBK - 1) / kDwBK : 0;
    if (nslices > 0) {
        if (moves_in) {
            for (int d = 0; d < kDwBK + 2 * p.halo; d += kDwBK) {
                load_row(lo - p.halo + d + mrow);
                put_row(ring, (d + mrow) & (kDwRing - 1));
            }
        } else {
            load_row(lo + mrow);
            put_row(delta(0), mrow);
            if (col_sums) { c0 = c0 + r0; c1 = c1 + r1; }
        }
        __syncthreads();
        for (int t = 0; t < nslices; ++t) {
            const bool more = t + 1 < nslices;
            if (more) load_row(lo + (t + 1) * kDwBK + (moves_in ? p.halo : 0) + mrow);
            const uint8_t* D = delta(t & 1);
            const int base = t * kDwBK + p.halo + (kh - 1) * W1 + frow;
#pragma unroll
            for (int s = 0; s < kDwBK / 16; ++s) {
                SplitFrag fd, fi[3];
                {
                    const uint8_t* a = D + half_addr(16 * s + frow, wj);
                    fd.hi = frag(a, a + 4 * kDwRow, 0);     // four rows on: the same bit 1, so the same half
                    fd.mid = frag(a, a + 4 * kDwRow, 1);
                    fd.lo = frag(a, a + 4 * kDwRow, 2);
                }
#pragma unroll
                for (int kw = 0; kw < 3; ++kw) {
                    const int row = base + 16 * s + kw - 1;
                    const uint8_t* a = ring + half_addr(row & (kDwRing - 1), wi);
                    const uint8_t* b = ring + half_addr((row + 4) & (kDwRing - 1), wi);
                    fi[kw].hi = frag(a, b, 0);
                    fi[kw].mid = frag(a, b, 1);
                    fi[kw].lo = frag(a, b, 2);
                }
                mfma_split(acc, low, fi, fd);
            }
            if (more) {
                if (moves_in) {
                    put_row(ring, ((t + 1) * kDwBK + 2 * p.halo + mrow) & (kDwRing - 1));
                } else {
                    put_row(delta((t + 1) & 1), mrow);
                    if (col_sums) { c0 = c0 + r0; c1 = c1 + r1; }
                }
            }
            __syncthreads();
        }
    }

    const int64_t n_w = (int64_t)9 * C * C;
    float* PART = p.partial + ((int64_t)split * p.groups + group) * (n_w + C);
    const int co = co0 + 32 * wj + lane % 32;
    auto element = [&](int kw, int r) { return ((int64_t)(3 * kh + kw) * C + ci0 + 32 * wi + 8 * (r / 4) + 4 * (lane / 32) + r % 4) * C + co; };
    auto inside = [&](int r) { return ci0 + 32 * wi + 8 * (r / 4) + 4 * (lane / 32) + r % 4 < C && co < C; };
    float odd = 0.0f;    // NaN once a sum is infinite or NaN
#pragma unroll
    for (int kw = 0; kw < 3; ++kw)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float v = split_sum(acc[kw][r], low[kw][r]);
            odd = __fmaf_rn(v, 0.0f, odd);
            if (inside(r)) PART[element(kw, r)] = v;
        }
    // An infinite or NaN input element has also been multiplied by the zeros that stand for the delta where there is no pixel
    // and past the range.  Where the wavefront's 32 input channels hold one in the range, its sums that are not finite are
    // formed again, over the range's pixels alone.
    if (__builtin_expect(__any(!(odd == 0.0f)), 0)) {
        const float* IN = p.in + (int64_t)group * p.s_in + ci0 + 32 * wi;
        const int64_t first = image_pixels_before(p, lo - p.halo), end = image_pixels_before(p, hi + p.halo);
        odd = 0.0f;
        for (int64_t q = first + lane / 32; q < end; q += 2)
            if (ci0 + 32 * wi + lane % 32 < C) odd = __fmaf_rn(IN[q * C + lane % 32], 0.0f, odd);
        if (__any(!(odd == 0.0f))) {
#pragma unroll 1
            for (int t = 0; t < 48; ++t) {
                const int kw = t / 16, r = t % 16;
                if (!inside(r) || __builtin_isfinite(PART[element(kw, r)])) continue;
                PART[element(kw, r)] = pixel_sum(p, group, lo, hi, 3 * kh + kw, ci0 + 32 * wi + 8 * (r / 4) + 4 * (lane / 32) + r % 4, co);
            }
        }
    }
    if (col_sums) {   // rows added in order (the operand tiles are no longer read)
        float* red = (float*)lds;
        if (!moves_in) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                red[mrow * 64 + mch + e] = c0[e];
                red[mrow * 64 + mch + 4 + e] = c1[e];
            }
        }
        __syncthreads();
        if (threadIdx.x < 64 && co0 + (int)threadIdx.x < C) {
            float sum = 0.0f;
            for (int r = 0; r < kDwBK; ++r) sum += red[r * 64 + threadIdx.x];
            PART[n_w + co0 + threadIdx.x] = sum;
        }
    }
}

bool aligned16(const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; }

// Rows of virtual pixels that a tile's nine taps can touch: its own span -- one zero column per image row it leaves, one
// zero row per image -- and one row and one column on either side.
int64_t strip_rows_of(int H, int W) {
    const int64_t step = kBM - 1;
    return kBM + (step + W - 1) / W + ((step + (int64_t)H * W - 1) / ((int64_t)H * W)) * (W + 1) + 2 * (W + 2);
}

template <int MODE>
hipError_t conv_launch(const ConvArgs& a, hipStream_t s) {
    if (a.groups < 1 || a.groups > 65535 || !conv3x3_split_fits(a.B, a.H, a.W, a.C)) return hipErrorInvalidValue;
    const uint8_t* w = MODE == 0 ? a.w_split : a.w_split_dx;
    if (!a.in || !w || !a.out || !aligned16(a.in) || !aligned16(w) || !aligned16(a.out) || !aligned16(a.residual) || !aligned16(a.mask)) return hipErrorInvalidValue;
    if (a.s_in % 4 || a.s_out % 4 || (a.residual && a.s_res % 4) || (a.mask && a.s_mask % 4)) return hipErrorInvalidValue;
    ConvSDev p = {};
    p.in = a.in; p.w = w; p.out = a.out; p.bias = a.bias; p.residual = a.residual; p.mask = a.mask;
    p.s_in = a.s_in; p.s_w = conv3x3_split_weight_bytes(1, a.C); p.s_out = a.s_out; p.s_bias = a.s_bias; p.s_res = a.s_res; p.s_mask = a.s_mask;
    p.groups = a.groups; p.B = a.B; p.H = a.H; p.W = a.W; p.C = a.C; p.P = a.B * a.H * a.W;
    p.relu = a.relu;
    if (MODE == 0 && a.stat_part) {
        if (a.C % kBN || !aligned16(a.stat_part)) return hipErrorInvalidValue;
        p.stat_part = a.stat_part;
    }
    p.strip_rows = (int)strip_rows_of(a.H, a.W);
    p.strip_bytes = std::max(p.strip_rows * kRow, kStageBytes);
    p.tiles_m = (p.P + kBM - 1) / kBM;
    p.tiles_n = (a.C + kBN - 1) / kBN;
    const int64_t total = (int64_t)a.groups * p.tiles_m * p.tiles_n;
    if (total > (1 << 30)) return hipErrorInvalidValue;
    p.total_tiles = (int)total;
    p.chunk = (int)((total + kXcds - 1) / kXcds);
    p.div_hw = make_div((unsigned)(a.H * a.W));
    p.div_w = make_div((unsigned)a.W);
    p.div_s = make_div((unsigned)((a.H + 1) * (a.W + 1)));
    p.div_w1 = make_div((unsigned)(a.W + 1));
    p.div_pg = make_div((unsigned)(p.tiles_m * p.tiles_n));
    p.div_tn = make_div((unsigned)p.tiles_n);
    const size_t lds = (size_t)p.strip_bytes + 3 * kSlice;
    void (*kern)(ConvSDev) = p.strip_rows <= 256 ? conv3x3_split_kernel<MODE, 4> : conv3x3_split_kernel<MODE, 5>;
    hipError_t e = ensure_dynamic_lds((const void*)kern, 160 * 1024);
    if (e != hipSuccess) return e;
    kern<<<(unsigned)(p.chunk * kXcds), kThreads, lds, s>>>(p);
    return hipGetLastError();
}

}  // namespace

bool conv3x3_split_fits(int B, int H, int W, int C) {
    if (B < 1 || H < 1 || W < 1 || C < 32 || C % kKC != 0 || C > 4096) return false;
    if (strip_rows_of(H, W) > kMaxStripRows || W + 2 > kDwMaxHalo) return false;
    // byte offsets of a group's tensor, and virtual pixel indices, stay below 2^31
    return (int64_t)B * H * W * C * 4 < ((int64_t)1 << 31) - ((int64_t)kBM * C * 4 + 65536) &&
           ((int64_t)B + 2) * (H + 1) * (W + 1) + kMaxStripRows < ((int64_t)1 << 31);
}

int64_t conv3x3_split_stat_parts(int B, int H, int W) { return ((int64_t)B * H * W + kBM - 1) / kBM; }

int64_t conv3x3_split_weight_bytes(int groups, int C) {
    return (int64_t)groups * (C / kKC) * ((C + kBN - 1) / kBN) * 9 * kSlice;
}

hipError_t launch_conv3x3_split_weights(const float* wa, const float* wb, uint8_t* fwd_a, uint8_t* fwd_b, uint8_t* dx_b, int64_t s_w,
                                        int groups, int C, hipStream_t s) {
    if (!wa || !wb || !fwd_a || !fwd_b || !dx_b || !aligned16(fwd_a) || !aligned16(fwd_b) || !aligned16(dx_b) || groups < 1 ||
        groups > 65535 || C < 32 || C % kKC != 0 || C > 4096)
        return hipErrorInvalidValue;
    SplitWeights p = {};
    p.w[0] = wa; p.w[1] = wb; p.w[2] = wb;
    p.dst[0] = fwd_a; p.dst[1] = fwd_b; p.dst[2] = dx_b;
    p.dx[2] = 1;
    p.s_w = s_w; p.s_dst = conv3x3_split_weight_bytes(1, C);
    p.C = C; p.tiles_n = (C + kBN - 1) / kBN;
    split_weights_kernel<<<dim3((unsigned)((C / kKC) * p.tiles_n * 9), (unsigned)groups, 3), 256, 0, s>>>(p);
    return hipGetLastError();
}

int conv3x3_split_dw_splits(int groups, int B, int H, int W, int C) {
    const int64_t V = (int64_t)B * (H + 1) * (W + 1);
    const int64_t blocks = (C + 63) / 64, tiles = groups * blocks * blocks;
    int64_t s = 256 / tiles;                           // one workgroup per compute unit (135 KB of LDS each), in one round
    const int64_t most = (V + 4 * kDwBK - 1) / (4 * kDwBK);   // at least four slices (sixteen: 59.5 against 24.9 us on 1 x 2 x 32 x 32 x 64)
    if (s > most) s = most;
    return s < 1 ? 1 : (int)s;
}

hipError_t launch_conv3x3_split_dw(const ConvArgs& a, hipStream_t s) {
    if (a.groups < 1 || a.groups > 65535 || !conv3x3_split_fits(a.B, a.H, a.W, a.C)) return hipErrorInvalidValue;
    if (!a.in || !a.dout || !a.partial || a.dw_splits < 1 || !a.g || !aligned16(a.in) || !aligned16(a.dout) || a.s_in % 4 || a.s_dout % 4) return hipErrorInvalidValue;
    ConvSDwDev p = {};
    p.in = a.in; p.dout = a.dout; p.partial = a.partial;
    p.s_in = a.s_in; p.s_dout = a.s_dout;
    p.groups = a.groups; p.B = a.B; p.H = a.H; p.W = a.W; p.C = a.C;
    p.V = a.B * (a.H + 1) * (a.W + 1);
    p.halo = a.W + 2;
    p.splits = a.dw_splits;
    p.k_chunk = (int)((((int64_t)p.V + p.splits - 1) / p.splits + kDwBK - 1) / kDwBK * kDwBK);
    p.blocks_n = (a.C + 63) / 64;
    p.tensor_bytes = (unsigned)a.B * a.H * a.W * 4u * (unsigned)a.C;
    p.div_s = make_div((unsigned)((a.H + 1) * (a.W + 1)));
    p.div_w1 = make_div((unsigned)(a.W + 1));
    const int64_t total = (int64_t)a.groups * p.splits * p.blocks_n * p.blocks_n;
    if (total > (1 << 30)) return hipErrorInvalidValue;
    p.total_tiles = (int)total;
    p.chunk = (int)((total + kXcds - 1) / kXcds);
    hipError_t e = ensure_dynamic_lds((const void*)conv3x3_split_dw_kernel, 160 * 1024);
    if (e != hipSuccess) return e;
    conv3x3_split_dw_kernel<<<(unsigned)(p.chunk * kXcds), kDwThreads, kDwRing * kDwRow + 2 * kDwBK * kDwRow, s>>>(p);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const ConvDwParts parts = {a.partial, a.g_w_off, a.g_b_off};
    return launch_conv_dw_finish(&parts, 1, p.splits, a.groups, a.C, a.g, a.ld, a.guest, s);
}

hipError_t launch_conv3x3_split_fwd(const ConvArgs& a, hipStream_t s) { return conv_launch<0>(a, s); }
hipError_t launch_conv3x3_split_dx(const ConvArgs& a, hipStream_t s) { return conv_launch<1>(a, s); }

}  // namespace ols
