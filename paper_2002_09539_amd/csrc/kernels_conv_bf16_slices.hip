// Forward and delta of the plain bf16 block in launches of middling size (see conv3x3_bf16_slices_fits): the same products as
// kernels_conv_bf16.hip in another structure.  One workgroup per 256 padded pixels x 64 output channels; the strip of input
// rows is copied to LDS through registers, and the nine taps' 64 x 64 kernel slices follow through two LDS buffers, a barrier per
// tap.  It moves more bytes (the delta reads the bf16 activations for its gate) but reads the kernels once per workgroup instead
// of once per wavefront, and in launches of middling size a whole step is up to 6 % faster, seen only under a sustained load
// (over the first milliseconds both are equal), where the unchanged kernel gradient beside it gains as well: what it saves is
// energy.  us per launch in a sustained run, 15 x 59 x 23 x 24 x 64, here / there: forward 45.8 / 52.3, with the tail 54.6 / 61.1,
// delta 49.8 / 49.7, kernel gradient beside it 43.9 / 45.9; at 16 x 128 x 32 x 32 x 64 208 / 187, 240 / 238, 214 / 179.
#include <type_traits>

#include "fast_div.h"
#include "gemm_bf16_tile.h"
#include "ols_internal.h"

namespace ols {

namespace {

constexpr int kThreads = kTileThreads;
constexpr int kXcds = 8;
constexpr int kCB = 64;     // channel block: contraction chunk and output-channel tile
constexpr int kBM = 256;    // padded pixels per tile

struct SliceDev {
    const uint16_t* in;      // FWD: layer input; DX: delta of the layer output   [groups][Pp][C] bf16
    const uint16_t* w;       // bf16 kernels [9][C][C]
    uint16_t* out;           // [Pp][C] (not with the fused tail)
    const float* bias;       // FWD
    const uint16_t* mask;    // DX: padded bf16 activations whose sign gates the result
    const float* xres;       // fused tail: the shortcut, fp32 [B H W][C]
    uint8_t* sign;           // fused tail: [Pp][C / 4] sign bytes
    float* pool_part;        // fused tail: [groups][tiles_m * 4 wavefronts][2][C] partial sums of the pooling
    int64_t s_x, s_sign, s_in, s_w, s_out, s_bias, s_mask;
    int B, H, W, C, Hp, Wp, Pp, halo;
    int tiles_m, tiles_n, total_tiles, chunk;
    FastDiv div_per, div_wp; // division by (H + 2) (W + 2) and by W + 2
    FastDiv div_pg, div_tn;  // division by tiles_m * tiles_n and by tiles_n
};

__device__ __forceinline__ int xcd_tile(int chunk, int total) {
    const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
    const int tile = xcd * chunk + slot;
    return (slot >= chunk || tile >= total) ? -1 : tile;
}

// padded pixel q -> is it an image pixel, and which (index in the unpadded [B H W] order)
__device__ __forceinline__ bool interior(const SliceDev& p, int q, int* unpadded) {
    const int per = p.Hp * p.Wp;
    const int n = (int)fast_div((unsigned)q, p.div_per), rem = q - n * per;
    const int y = (int)fast_div((unsigned)rem, p.div_wp), x = rem - y * p.Wp;
    *unpadded = (n * p.H + (y - 1)) * p.W + (x - 1);
    return y >= 1 && y <= p.H && x >= 1 && x <= p.W;
}

// ---------------------------------------------------------------------------------------------
// forward (MODE 0) and back-propagated delta (MODE 1)
// ---------------------------------------------------------------------------------------------
// LDS of the forward / delta kernel, in bf16 elements: the strip and two kernel slices -- or, if larger, the fp32 output
// staging of the four wavefronts (BM / 4 rows of 64 + 4 floats each), which takes their place after the last tap.
constexpr int kStagePitchF32 = kCB + 4;
enum { kOutBf16 = 0, kOutTail = 1 };
template <int BM, int OUT>
__host__ __device__ constexpr int conv_main_elems(int strip_rows, int slice_elems) {
    const int work = strip_rows * (kCB + 8) + 2 * slice_elems;
    const int stage = OUT != kOutBf16 ? BM * kStagePitchF32 * 2 : 0;
    return work > stage ? work : stage;
}

// NV: strip vectors per lane (upper bound of (BM + 2 halo) * 8 / 256); BM: pixels per tile.
template <int MODE, int OUT, int NV, int BM>
__global__ __launch_bounds__(kThreads, 2) void conv3x3_bf16_slices_kernel(SliceDev p) {
    using TB = typename std::conditional<MODE == 0, TileRC<kCB, kCB>, TileKC<kCB, kCB>>::type;   // FWD w[k = ci][n = co]; DX w[n = ci][k = co]
    constexpr int SP = kCB + 8;                  // strip pitch (bf16 elements): 144 bytes, conflict-free 16-byte reads
    constexpr int TM = BM / 128, TN = 2, KS = kCB / 16; // a wavefront owns BM / 4 pixels x 64 channels
    static_assert(TB::kLineStep == 32 && TB::kPerThread == 2, "a lane's vectors are 32 rows apart in the strip and in a kernel slice");
    extern __shared__ __attribute__((aligned(16))) uint16_t lds_all[];
    constexpr int kStripRows = NV * 32;          // every lane moves NV vectors: rows past BM + 2 halo are loaded and never read
    uint16_t* strip = lds_all;
    uint16_t* lds_b0 = lds_all + kStripRows * SP;
    auto lds_b = [&](int buf) { return lds_b0 + buf * TB::kElems; };
    // the fp32 output is staged over the strip and the kernel slices together (conv_main_elems)
    uint8_t* row_flag = (uint8_t*)(lds_all + conv_main_elems<BM, OUT>(kStripRows, TB::kElems));   // [BM] 1: image pixel, 0: border
    int* row_up = (int*)row_flag;   // fused tail / unpadded output instead: [BM] the pixel's index in the unpadded [B H W] order, -1 for the border

    const int tile = xcd_tile(p.chunk, p.total_tiles);
    if (tile < 0) return;
    const int per_group = p.tiles_m * p.tiles_n;
    const int group = (int)fast_div((unsigned)tile, p.div_pg);
    const int in_group = tile - group * per_group;
    const int tm = (int)fast_div((unsigned)in_group, p.div_tn), tn = in_group - tm * p.tiles_n;
    const int m0 = tm * BM, n0 = tn * kCB;
    const uint16_t* IN = p.in + (int64_t)group * p.s_in;
    const uint16_t* Wg = p.w + (int64_t)group * p.s_w;
    const int C = p.C;

    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int lane32 = lane % 32, half = lane / 32;
    const int wm0 = wave * (BM / 4);

    // Byte offsets in a [rows][C] bf16 tensor: lane t of the workgroup owns the 16-byte vector t % 8 of row t / 8, and its
    // further vectors lie 32 rows below.  The same lane offset serves the strip and the kernel slices.
    const unsigned row_bytes = 2u * (unsigned)C;
    const unsigned lane_off = (threadIdx.x / 8) * row_bytes + (threadIdx.x % 8) * 16u;
    const unsigned step32 = 32u * row_bytes;
    const rsrc_t in_rs = make_rsrc(IN, (unsigned)p.Pp * row_bytes);
    const rsrc_t w_rs = make_rsrc(Wg, 9u * (unsigned)C * row_bytes);
    // rows m0 - halo .. of channels c0 .. c0 + 63: rows before the tensor wrap to offsets beyond its end, rows after it
    // lie beyond it too -- both read as zeros.  Every lane requests all its vectors at once (one round trip), then
    // writes them to LDS.
    const unsigned strip_off = (unsigned)(m0 - p.halo) * row_bytes + lane_off;
    uint16_t* strip_lane = strip + (threadIdx.x / 8) * SP + (threadIdx.x % 8) * 8;
    auto load_strip = [&](u4 (&r)[NV], int c0) {
#pragma unroll
        for (int t = 0; t < NV; ++t) r[t] = buf_load(in_rs, strip_off + t * step32, 2u * c0);
    };
    auto store_strip = [&](const u4 (&r)[NV]) {
#pragma unroll
        for (int t = 0; t < NV; ++t) *(u4*)(strip_lane + t * 32 * SP) = r[t];
    };
    // the 64 x 64 kernel slice of one tap.  Memory [ci][co]: FWD (row-contiguous tile) k = ci, rows = co; DX
    // (K-contiguous tile) rows = ci, k = co
    auto load_b = [&](u4 (&r)[TB::kPerThread], int tap, int c0) {
        const unsigned first = 2u * (unsigned)((tap * C + (MODE == 0 ? c0 : n0)) * C + (MODE == 0 ? n0 : c0));
#pragma unroll
        for (int t = 0; t < TB::kPerThread; ++t) r[t] = buf_load(w_rs, lane_off + t * step32, first);
    };
    auto store_b = [&](int buf, const u4 (&r)[TB::kPerThread]) {
        uint16_t* dst = TB::lane_lds(lds_b(buf));
#pragma unroll
        for (int t = 0; t < TB::kPerThread; ++t) *(u4*)(dst + t * TB::kLdsLineStep) = r[t];
    };

    // The MFMA takes the KERNEL fragment first and the pixel fragment second, so the accumulator tile is out^T:
    // register r of a lane holds pixel lane % 32 and channel 8 (r / 4) + 4 (lane / 32) + r % 4 of its 32 x 32 block --
    // four consecutive channels per register quad, which the epilogue packs and stores as one piece.
    f16v acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    bf16x8 fa[2][TM], fb[2][TN];
    auto load_frags = [&](int buf, const uint16_t* a_base, const uint16_t* b_tile, int s) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
            fa[buf][i] = __builtin_bit_cast(bf16x8, *(const u4*)(a_base + (wm0 + 32 * i + lane32) * SP + 16 * s + 8 * half));
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[buf][j] = TB::frag(b_tile, 32 * j, s, lane);
    };
    auto mfmas = [&](int buf) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[buf][j], fa[buf][i], acc[i][j], 0, 0, 0);
    };

    // Kernel slices travel kAhead taps ahead of their use (a tap's 16 MFMAs per wavefront are shorter than a round trip
    // to L2): a ring of kAhead register sets, slice t in set t % kAhead.
    constexpr int kAhead = 3;
    u4 rb[kAhead][TB::kPerThread];
    // Delta: the activations whose sign gates the result -- the 16-byte vectors of the wavefront's own rows that this
    // lane will write -- are requested kMaskTap taps into a chunk, when no kernel slice is in flight any more (with the
    // long strips of wide images the registers do not allow it: there they are requested after the last tap).
    constexpr int kVecB = kCB / 8, kPerB = (BM / 4) * kVecB / 64, kMaskTap = NV <= 12 ? 6 : 9;
    u4 mk[MODE == 1 && OUT == kOutBf16 ? kPerB : 1];
    const uint16_t* Mk = MODE == 1 && p.mask ? p.mask + (int64_t)group * p.s_mask : nullptr;
    const rsrc_t mk_rs = make_rsrc(Mk ? Mk : IN, Mk ? (unsigned)p.Pp * row_bytes : 0u);
    // the wavefront's own rows of the [Pp][C] bf16 output: lane l moves the vector l % 8 of rows wm0 + l / 8 + 8 t
    const unsigned own_off = (unsigned)(m0 + wm0 + lane / kVecB) * row_bytes + 2u * (unsigned)n0 + (lane % kVecB) * 16u;
    const unsigned step8 = (64 / kVecB) * row_bytes;
    auto load_mask = [&]() {
#pragma unroll
            for (int t = 0; t < kPerB; ++t) mk[t] = buf_load(mk_rs, own_off + t * step8, 0u);
    };
    // Forward: the lane's channels of the bias (register quad g4 of block j: channels 32 j + 8 g4 + 4 (lane / 32) ..),
    // requested at the same point and added in the epilogue.
    f4 bq[MODE == 0 ? TN : 1][4];
    // (an empty range without a bias: zeros, and no branch for the waits on the kernel slices to be merged over)
    const rsrc_t bias_rs = make_rsrc(MODE == 0 && p.bias ? (const void*)(p.bias + (int64_t)group * p.s_bias + n0) : (const void*)IN,
                                     MODE == 0 && p.bias ? kCB * 4u : 0u);
    auto load_bias = [&]() {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) bq[j][g4] = __builtin_bit_cast(f4, buf_load(bias_rs, 16u * half + 128u * j + 32u * g4, 0u));
    };
    // Fused tail: the shortcut's fp32 rows that this lane will add (vector l % 16 of the unpadded rows behind the
    // wavefront's padded rows l / 16 + 4 t) -- the first batch of eight is requested at the same point, the second in
    // the epilogue while the first is consumed.
    constexpr int kTailBatch = 8;
    f4 xpre[OUT == kOutTail ? kTailBatch : 1];
    int up_pre[OUT == kOutTail ? kTailBatch : 1];
    const rsrc_t x_rs = make_rsrc(OUT == kOutTail ? (const void*)(p.xres + (int64_t)group * p.s_x) : (const void*)IN,
                                  OUT == kOutTail ? (unsigned)(p.B * p.H * p.W) * 2u * row_bytes : 0u);
    auto load_shortcut = [&]() {
        if constexpr (OUT == kOutTail) {
#pragma unroll
            for (int t = 0; t < kTailBatch; ++t) up_pre[t] = row_up[wm0 + lane / (kCB / 4) + 4 * t];
#pragma unroll
            for (int t = 0; t < kTailBatch; ++t)   // border rows: -1 wraps to an offset beyond the tensor, zeros come back
                xpre[t] = __builtin_bit_cast(f4, buf_load(x_rs, (unsigned)up_pre[t] * 2u * row_bytes + 4u * n0 + (lane % (kCB / 4)) * 16u, 0u));
        }
    };
    for (int c0 = 0; c0 < C; c0 += kCB) {
        // the previous chunk's last barrier has passed: nobody reads the strip or the kernel buffers any more
        {
            u4 rs[NV];
            load_b(rb[0], 0, c0);   // what the first tap needs goes first
            load_strip(rs, c0);
#pragma unroll
            for (int t = 1; t < kAhead; ++t) load_b(rb[t], t, c0);
            if (c0 == 0) {
                int up;   // which rows of the tile are image pixels (the others get the zero border)
                const int q = m0 + threadIdx.x;
                const bool img = q < p.Pp && interior(p, q, &up);
                if (threadIdx.x < BM) {
                    if constexpr (OUT == kOutTail) row_up[threadIdx.x] = img ? up : -1; else row_flag[threadIdx.x] = img ? 1 : 0;
                }
            }
            store_b(0, rb[0]);
            store_strip(rs);
        }
        __syncthreads();
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            if (tap + kAhead < 9) load_b(rb[tap % kAhead], tap + kAhead, c0);   // its slice is in LDS already
            if (tap == kMaskTap) {   // in every chunk: a branch here would make the waits on the kernel slices wait for these too
                if constexpr (MODE == 1) load_mask(); else load_bias();
                load_shortcut();
            }
            const int dy = tap / 3 - 1, dx = tap % 3 - 1;
            const int shift = (MODE == 0 ? 1 : -1) * (dy * p.Wp + dx);
            const uint16_t* a_base = strip + (p.halo + shift) * SP;
            const uint16_t* b_tile = lds_b(tap & 1);
            load_frags(0, a_base, b_tile, 0);
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if (s + 1 < KS) load_frags((s + 1) & 1, a_base, b_tile, s + 1);
                __builtin_amdgcn_sched_barrier(0);
                mfmas(s & 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (tap + 1 < 9) store_b((tap + 1) & 1, rb[(tap + 1) % kAhead]);
            __syncthreads();
        }
    }

    if (kMaskTap >= 9) {
        if constexpr (MODE == 1) load_mask(); else load_bias();
        load_shortcut();
    }
    // Epilogue: the tile goes through LDS (the strip's place) so that every lane then moves 16-byte vectors.
    if constexpr (OUT == kOutTail) {
        // a2 = relu(convolution + bias + shortcut) on the image pixels: its sign bytes and, per wavefront (64 consecutive
        // padded pixels, which touch at most two samples because a padded image has at least 64), the channel sums of its
        // rows in the first and in the second of those samples.  A later pass adds the wavefronts' sums per sample in
        // wavefront order.  Staging as for the fp32 output; lane l then owns the channel quad l % 16 of rows l / 16 + 4 t.
        constexpr int FP = kStagePitchF32, WR = BM / 4;
        constexpr int kVecPerRow = kCB / 4, kPer = WR * kVecPerRow / 64, kBatch = kTailBatch;
        static_assert(WR == 64, "the partial sums are kept per 64 rows");
        float* stage = (float*)lds_all + wave * WR * FP;
        const int r0 = lane / kVecPerRow, cq = lane % kVecPerRow;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    const f4 o = {acc[i][j][4 * g4] + bq[j][g4][0], acc[i][j][4 * g4 + 1] + bq[j][g4][1], acc[i][j][4 * g4 + 2] + bq[j][g4][2],
                                  acc[i][j][4 * g4 + 3] + bq[j][g4][3]};
                    *(f4*)(stage + (32 * i + lane32) * FP + 32 * j + 8 * g4 + 4 * half) = o;
                }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int q0 = m0 + wm0;                                    // the wavefront's first padded pixel
        const int per = p.Hp * p.Wp;
        const int next_sample = ((int)fast_div((unsigned)q0, p.div_per) + 1) * per;   // first pixel of the second sample
        const rsrc_t sg_rs = make_rsrc(p.sign + (int64_t)group * p.s_sign, (unsigned)p.Pp * (unsigned)(C / 4));
        f4 sum0 = {0.f, 0.f, 0.f, 0.f}, sum1 = {0.f, 0.f, 0.f, 0.f};
        static_assert(kPer == 2 * kBatch, "two batches of shortcut rows per lane");
        f4 xnext[kBatch];
        int up_next[kBatch];
#pragma unroll
        for (int t = 0; t < kBatch; ++t) up_next[t] = row_up[wm0 + r0 + 4 * (kBatch + t)];
#pragma unroll
        for (int t = 0; t < kBatch; ++t)   // the second batch travels while the first is consumed
            xnext[t] = __builtin_bit_cast(f4, buf_load(x_rs, (unsigned)up_next[t] * 2u * row_bytes + 4u * n0 + cq * 16u, 0u));
#pragma unroll
        for (int t0 = 0; t0 < kPer; t0 += kBatch) {
            f4 yv[kBatch], xv[kBatch];
            int up[kBatch];
#pragma unroll
            for (int t = 0; t < kBatch; ++t) {
                up[t] = t0 == 0 ? up_pre[t] : up_next[t];
                xv[t] = t0 == 0 ? xpre[t] : xnext[t];
            }
#pragma unroll
            for (int t = 0; t < kBatch; ++t) yv[t] = *(const f4*)(stage + (r0 + 4 * (t0 + t)) * FP + cq * 4);
#pragma unroll
            for (int t = 0; t < kBatch; ++t) {
                const int q = q0 + r0 + 4 * (t0 + t);
                const bool img = up[t] >= 0;
                unsigned bits = 0;
                f4 a;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    a[e] = img ? fmaxf(yv[t][e] + xv[t][e], 0.0f) : 0.0f;
                    bits |= a[e] > 0.0f ? (1u << e) : 0u;
                }
                if (q < next_sample) sum0 = sum0 + a; else sum1 = sum1 + a;
                __builtin_amdgcn_raw_buffer_store_b8((unsigned char)bits, sg_rs, (int)((unsigned)q * (unsigned)(C / 4) + n0 / 4 + cq), 0, 0);   // rows past the tensor are dropped
            }
        }
        // the four lanes of a channel quad, in lane order, through the staging area (all its reads are done)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        f4* red = (f4*)stage;
        red[lane] = sum0;
        red[64 + lane] = sum1;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (lane < 2 * kVecPerRow) {   // lanes 0 .. 15: first sample, 16 .. 31: second
            const f4* r = red + 64 * (lane / kVecPerRow) + lane % kVecPerRow;
            const f4 o = ((r[0] + r[16]) + r[32]) + r[48];
            float* PP = p.pool_part + ((((int64_t)group * p.tiles_m + tm) * 4 + wave) * 2 + lane / kVecPerRow) * C + n0;
            *(f4*)(PP + 4 * (lane % kVecPerRow)) = o;
        }
    } else {
        // wavefront-local as well: a wavefront stages and moves its own BM / 4 rows
        const rsrc_t out_rs = make_rsrc((const uint16_t*)p.out + (int64_t)group * p.s_out, (unsigned)p.Pp * row_bytes);
        uint16_t* stage = lds_all + wm0 * SP;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[e] = acc[i][j][4 * g4 + e];
                        if constexpr (MODE == 0) v[e] = fmaxf(v[e] + bq[j][g4][e], 0.0f);
                    }
                    u2 o;   // round to nearest even (v_cvt_pk_bf16_f32)
                    o.x = __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{v[0], v[1]}, bf16x2));
                    o.y = __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{v[2], v[3]}, bf16x2));
                    *(u2*)(stage + (32 * i + lane32) * SP + 32 * j + 8 * g4 + 4 * half) = o;
                }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        u4 val[kPerB];
#pragma unroll
        for (int t = 0; t < kPerB; ++t) {
            const int v = lane + t * 64;
            val[t] = *(const u4*)(stage + (v / kVecB) * SP + (v % kVecB) * 8);
        }
#pragma unroll
        for (int t = 0; t < kPerB; ++t) {
            u4 o = val[t];
            if (MODE == 0) {
                if (!row_flag[wm0 + (lane + t * 64) / kVecB]) o = u4{0u, 0u, 0u, 0u};   // the zero border the next layer relies on
            } else if (Mk) {
#pragma unroll
                for (int w = 0; w < 4; ++w) {   // a bf16 is positive iff its bits are in [0x0001, 0x7FFF]
                    const unsigned int lo = mk[t][w] & 0xFFFFu, hi = mk[t][w] >> 16;
                    const unsigned int keep = ((lo - 1u) < 0x7FFFu ? 0xFFFFu : 0u) | ((hi - 1u) < 0x7FFFu ? 0xFFFF0000u : 0u);
                    o[w] &= keep;
                }
            }
            buf_store(o, out_rs, own_off + t * step8);   // rows past the tensor are dropped
        }
    }
}

bool aligned16(const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; }

template <int MODE>
hipError_t slices_launch(const ConvBArgs& a, hipStream_t s) {
    const bool tail = MODE == 0 && a.tail;
    if (a.groups < 1 || a.groups > 65535 || a.B < 1 || a.H < 1 || a.W < 1 || a.W > kConvBf16MaxWidth || a.C < kCB || a.C % kCB != 0 || a.C > 1024)
        return hipErrorInvalidValue;
    // 32-bit byte offsets inside one group's bf16 tensor, with room for the rows a tile's strip reaches past either end
    if ((int64_t)a.B * (a.H + 2) * (a.W + 2) * a.C >= ((int64_t)1 << 31) - (int64_t)1024 * a.C) return hipErrorInvalidValue;
    if (!a.in || !a.w || !aligned16(a.in) || !aligned16(a.w) || a.s_in % 8 || a.s_w % 8) return hipErrorInvalidValue;
    if (a.out_f32 || a.out_unpadded || a.stat_part) return hipErrorInvalidValue;
    if (!tail && (!a.out || !aligned16(a.out) || a.s_out % 8)) return hipErrorInvalidValue;
    if (MODE == 0 && (!a.bias || !aligned16(a.bias) || a.s_bias % 4 || (tail ? a.relu : !a.relu))) return hipErrorInvalidValue;
    if (MODE == 1 && (!a.mask || !aligned16(a.mask) || a.s_mask % 8)) return hipErrorInvalidValue;
    if (tail) {   // 16-byte vectors of the shortcut, 32-bit byte offsets in it, at most two samples per 64 padded pixels
        if (!a.xres || !a.sign || !a.pool_part || !aligned16(a.xres) || !aligned16(a.pool_part) || a.s_x % 4 ||
            (a.H + 2) * (a.W + 2) < 64 || (int64_t)a.B * a.H * a.W * a.C >= ((int64_t)1 << 30) - 1024)
            return hipErrorInvalidValue;
    }
    SliceDev p = {};
    p.in = (const uint16_t*)a.in; p.w = (const uint16_t*)a.w; p.out = (uint16_t*)a.out;
    p.bias = a.bias; p.mask = (const uint16_t*)a.mask; p.xres = a.xres; p.sign = a.sign; p.pool_part = a.pool_part;
    p.s_x = a.s_x; p.s_sign = a.s_sign; p.s_in = a.s_in; p.s_w = a.s_w; p.s_out = a.s_out; p.s_bias = a.s_bias; p.s_mask = a.s_mask;
    p.B = a.B; p.H = a.H; p.W = a.W; p.C = a.C;
    p.Hp = a.H + 2; p.Wp = a.W + 2; p.Pp = a.B * p.Hp * p.Wp; p.halo = p.Wp + 1;
    p.div_per = make_div((unsigned)(p.Hp * p.Wp));
    p.div_wp = make_div((unsigned)p.Wp);
    p.tiles_m = (p.Pp + kBM - 1) / kBM;
    p.tiles_n = a.C / kCB;
    p.div_pg = make_div((unsigned)(p.tiles_m * p.tiles_n));
    p.div_tn = make_div((unsigned)p.tiles_n);
    const int64_t total = (int64_t)a.groups * p.tiles_m * p.tiles_n;
    if (total > (1 << 30)) return hipErrorInvalidValue;
    p.total_tiles = (int)total;
    p.chunk = (int)((total + kXcds - 1) / kXcds);
    const size_t b_elems = MODE == 0 ? TileRC<kCB, kCB>::kElems : TileKC<kCB, kCB>::kElems;
    constexpr int NV0 = ((kBM + 2 * 35) * (kCB / 8) + kThreads - 1) / kThreads;                        // widths up to 32
    constexpr int NV1 = ((kBM + 2 * (kConvBf16MaxWidth + 3)) * (kCB / 8) + kThreads - 1) / kThreads;   // any width
    const int nv = ((kBM + 2 * p.halo) * (kCB / 8) + kThreads - 1) / kThreads;
    if (nv > NV1) return hipErrorInvalidValue;
    const int lds_rows = 32 * (nv <= NV0 ? NV0 : NV1);   // the kernel's strip holds all the vectors its lanes move
    const size_t main_elems = tail ? conv_main_elems<kBM, kOutTail>(lds_rows, (int)b_elems) : conv_main_elems<kBM, kOutBf16>(lds_rows, (int)b_elems);
    const size_t lds = main_elems * sizeof(uint16_t) + (tail ? kBM * sizeof(int) : kBM);   // strip and kernel slices (or the fp32 staging), row flags / indices
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    auto pick = [&](auto narrow) -> void (*)(SliceDev) {
        constexpr int NV = decltype(narrow)::value;
        if constexpr (MODE == 1) return conv3x3_bf16_slices_kernel<1, kOutBf16, NV, kBM>;
        else return tail ? conv3x3_bf16_slices_kernel<0, kOutTail, NV, kBM> : conv3x3_bf16_slices_kernel<0, kOutBf16, NV, kBM>;
    };
    void (*kern)(SliceDev) = nv <= NV0 ? pick(std::integral_constant<int, NV0>()) : pick(std::integral_constant<int, NV1>());
    if (lds > 64 * 1024) {
        hipError_t e = ensure_dynamic_lds((const void*)kern, 160 * 1024);
        if (e != hipSuccess) return e;
    }
    kern<<<(unsigned)(p.chunk * kXcds), kThreads, lds, s>>>(p);
    return hipGetLastError();
}

}  // namespace

// The rule, from whole steps of 74 plain blocks on either path, by tiles of 512 pixels x 64 channels (us for two rounds, there /
// here).  64 channels: 192 tiles 258 / 261, 200 271 / 267, 220 549 / 527; 264 896 / 914, 308 319 / 320, 330 326 / 325; 512 816 / 806,
// 574 916 / 885, 960 1896 / 1815, 1125 740 / 697, 1504 2614 / 2542, 2260 2528 / 2477, 2604 2875 / 2806; 3542 3610 / 3674, 4624 4660 /
// 4790.  128 channels: 224 384 / 370, 340 875 / 860, 368 1357 / 1305; 480 1060 / 1075, 656 1334 / 1346, 1808 2955 / 3054.  192: 90 560
// / 586, 144 666 / 706, 225 822 / 815, 288 1004 / 1025, 384 1143 / 1102 and 1178 / 1142, 684 1830 / 1880.  256, never taken: 112 646 / 676,
// 160 798 / 858, 256 1053 / 1038, 272 1089 / 1163, 324 1211 / 1243, 512 1677 / 1747, 992 2809 / 2945.  Fewer tiles: there by 1 to 7 %.
bool conv3x3_bf16_slices_fits(int groups, int B, int H, int W, int C) {
    const int64_t tiles = (int64_t)groups * (((int64_t)B * (H + 2) * (W + 2) + 511) / 512) * (C / kCB);
    if ((H + 2) * (W + 2) < 64) return false;   // (the unfused tail needs the fp32 output)
    if (C > 192) return false;
    return C == kCB ? (tiles >= 200 && tiles <= 256) || (tiles >= 500 && tiles <= 3072) : tiles >= 200 && tiles <= 400;
}
hipError_t launch_conv3x3_bf16_slices_fwd(const ConvBArgs& a, hipStream_t s) { return slices_launch<0>(a, s); }
hipError_t launch_conv3x3_bf16_slices_dx(const ConvBArgs& a, hipStream_t s) { return slices_launch<1>(a, s); }

}  // namespace ols
