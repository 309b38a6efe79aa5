// 3 x 3 convolutions (stride 1, zero padding 1) of the per-worker residual block with bf16 operands and fp32
// accumulation on the matrix cores (v_mfma_f32_32x32x16_bf16), grouped over the m workers: forward, back-propagated
// delta, kernel / bias gradient; plus the conversion of the input batch, the block's tail (shortcut, ReLU, pooling) and
// the pooling backward.  The model is the first residual stage of the network of Section 4 (arXiv 2002.09539,
// "Experimental setting") and produces the stochastic gradients g_i of Section 2; every tensor is rounded to bf16 (to
// nearest even) where it becomes an operand of a convolution's products, sums and everything else stay fp32.
//
// Layout: the bf16 operand tensors are stored WITH their zero border, [group][Pp][C] with Pp = B (H + 2) (W + 2) padded
// pixels in (sample, row, column) order and the channel contiguous.  A tap (kh, kw) is then the same shift
// s = (kh - 1) (W + 2) + (kw - 1) of the pixel index for every pixel, so
//   FWD  out[q][co] = sum_{tap, ci} in[q + s_tap][ci] w[tap][ci][co]
//   DX   din[q][ci] = sum_{tap, co} dout[q - s_tap][co] w[tap][ci][co]
//   DW   dw[tap][ci][co] = sum_q in[q + s_tap][ci] dout[q][co]
// are plain GEMMs over shifted row windows with no per-pixel case analysis: interior pixels only ever reach their own
// image's border, and every producer writes zeros to the border positions (the forward epilogue explicitly, the gates of
// the backward pass by themselves, because a zero activation gates its delta).  Rows outside [0, Pp) are read as zeros.
//
// FWD / DX: one workgroup per 512 padded pixels x 64 output channels (256 x 64 or 256 x 32 in small launches, see conv_tile).
// The input rows m0 - (W + 3) .. m0 + 512 + (W + 3) of a 64-channel chunk are loaded straight into LDS ONCE (a strip); the nine
// taps read their pixel fragments from it at nine row offsets.  The kernels' fragments come from a copy in fragment order that
// is made once per step (kernel_images, in the launch that converts the batch) straight into registers, four steps of 16
// channels ahead: no barrier between the taps.  Four wavefronts of 128 x 64; the MFMA takes the kernel fragment first, so a
// lane's accumulators are four consecutive channels of one pixel, packed by the hardware conversion and staged through LDS for
// 16-byte stores; every wavefront stages and stores its own rows, 64 at a time, so the epilogue has no workgroup barrier.
// The second convolution's epilogue is the block's tail: it adds the shortcut, applies the ReLU, keeps the activation's sign
// (one bit per element) for the backward pass and channel sums per 64 pixels for the pooling -- neither the convolution's output
// nor the activation is ever stored.  (Images of fewer than 64 padded pixels take the unfused route: conv + bias in fp32, then
// one streaming pass.)
// DW: one workgroup per (pixel range, 64 x 64 block of input x output channels); each of twelve wavefronts holds the
// three taps of a kernel row over 32 x 64 channels (96 registers per lane) for half of the contraction steps; per 96
// pixels 96 new input rows enter a ring of LDS rows (read with the transpose load at nine row offsets) and 96 delta rows a
// pair of buffers; ranges are summed in range order by the finish pass shared with the fp32 kernels (no atomics).
// All three address global memory through buffer descriptors: the hardware's range check returns zeros for the rows a
// strip reaches past either end of the tensor and drops the stores of a last tile's missing rows, so the loads and stores
// carry no per-lane predicates, selects or 64-bit address arithmetic.
//
// Measured at the benchmark shape (16 workers x 128 samples x 32 x 32 x 64 channels, 154.6 GFLOP per launch), us per launch within
// a step, before (256 x 64 tiles, kernel slices through LDS with a barrier per tap, the strip through registers) and now:
// forward with bf16 out 208 and 187 (180 without the sign bytes that it now leaves), forward with fp32 out 231 and 205, delta
// with bf16 out 214 and 179, with fp32 out 235 and 196 (206 and 240 while it read the bf16 activations for their sign: 0.3 GB
// instead of 34 MB), forward with the fused tail 240 and 238; 3 x 20 x 13 x 15 x 128 alone, bf16 out, 12.1 and 7.9.
// What bounds FWD / DX: energy.  Alone on the same inputs forward (bf16 out) takes 218 us; its taps without loads and epilogue
// 108, everything but the taps 122 (0.64 GB at 5.3 TB/s): the two add although two workgroups share a compute unit.  With all
// operands zero the whole takes 155 and the taps 87, and three other structures end at the same time: eight wavefronts that walk
// tiles with their half of the kernel in 144 registers and the next strip on its way (231, its taps alone 136: 64 x 32 per
// wavefront is bound by LDS reads), the same as two workgroups of four wavefronts (224), and four wavefronts with the whole
// kernel in 288 registers (one per SIMD, the epilogue in the open; 14 % slower than eight).
// The shortcut rows of the fused tail (fp32, 16 vectors per lane and half) are requested in batches of eight, the first two taps
// before the end and each further one while the batch before it is consumed (two batches ahead: no change); of four in the
// smaller tiles, where that leaves the registers of a third workgroup per compute unit (steps of 36 blocks 0.3 % faster on average, up to 0.9 %).
// The kernel gradient had four wavefronts of 32 x 32 channels x nine taps, two workgroups per compute unit, 64 pixels and
// a strip of 64 + 2 (W + 3) rows per slice: 170 us + 14 for the finish pass alone, 198 + 15 in a whole step.  Now 160 + 9
// and 185 + 9: the ring fetches a row once instead of 2.1 times, the taps of a kernel row share three transpose reads
// (seven reads feed six products, from twenty for nine), slices are requested two ahead, and the halves of the steps meet
// in LDS, so that there are half as many partial sums.  Without its loads it takes 168 us in a step, without its fragment
// reads 167, with one product of six 129: no single one bounds it, what is left is their overlap at 2.0 GHz.  The
// descriptor and the choice of its tensor have to be in scalar registers: with a per-lane choice the compiler loops over
// the lanes of every load (193).  Not kept: eight wavefronts with nine taps each, every fragment read a kernel row ahead
// and across the slice's barrier (212); two workgroups of six wavefronts, 48 pixels per slice (232).
// Tried and not kept: in the kernel gradient two slices of loads in flight (400 registers, one wavefront per SIMD: 349 us),
// fragment reads two kernel rows ahead (259 against 258 us); in forward / delta a raised wavefront priority (s_setprio)
// outside or inside the tap loop (+-1 %), the bias loaded straight into the accumulators before the first tap, the first
// MFMAs of a tile with a zero third operand instead of cleared accumulators (no change).
#include <algorithm>
#include <type_traits>

#include "fast_div.h"
#include "gemm_bf16_tile.h"
#include "ols_internal.h"

namespace ols {

// Measurement builds only (-DOLS_CONV_PHASE_PROBE): lane 0 of every forward / delta workgroup leaves s_memrealtime
// readings (100 MHz) at six points of its tile, which ols_debug_conv_phases() copies out.  [kernel: 0 forward with
// bf16 output, 1 forward with another output, 2 delta][tile][point].  Without the flag nothing of this exists.
#ifdef OLS_CONV_PHASE_PROBE
constexpr int kProbeTiles = 16384;
__device__ unsigned long long conv_phase_probe[3][kProbeTiles][8];
#define OLS_TP(k)                                                                                             \
    do {                                                                                                      \
        if (threadIdx.x == 0 && tile < kProbeTiles)                                                           \
            conv_phase_probe[MODE == 1 ? 2 : (OUT == kOutBf16 ? 0 : 1)][tile][k] = wall_clock64();            \
    } while (0)
#else
#define OLS_TP(k) do { } while (0)
#endif

namespace {

constexpr int kThreads = kTileThreads;
constexpr int kXcds = 8;
constexpr int kCB = 64;     // channel block: contraction chunk and output-channel tile
typedef __attribute__((address_space(3))) void* lds_void_ptr;
constexpr int kDwBK = 96;   // padded pixels per slice of the kernel-gradient contraction

struct ConvBDev {
    const uint16_t* in;      // FWD: layer input; DX: delta of the layer output; DW: layer input   [groups][Pp][C] bf16
    const uint16_t* w;       // FWD, DX: bf16 kernels in fragment order (see kernel_images)
    const uint16_t* dout;    // DW: delta of the layer output
    const uint16_t *in_b, *dout_b;   // DW of two layers: the second's, after `layer_tiles` tiles
    float* partial_b;
    int layer_tiles;
    void* out;               // FWD, DX: [Pp][C], bf16 or fp32
    const float* bias;       // FWD
    uint8_t* gate;           // sign bytes, one per row of the output and four channels: DX, they gate the result; FWD with bf16
                             // output, it leaves its own
    float* partial;          // DW
    const float* xres;       // FWD with the fused tail: the shortcut, fp32 [B H W][C]
    uint8_t* sign;           // FWD with the fused tail: [Pp][C / 4] sign bytes
    float* pool_part;        // FWD with the fused tail: [groups][units][2][C] partial sums of the pooling
    float* stat_part;        // FWD with the unpadded fp32 output, optional: [groups][units][3][C]
                             // statistics of the output's image pixels (count, mean, sum of squared deviations)
    int64_t s_x, s_sign;
    int64_t s_in, s_w, s_dout, s_out, s_bias, s_gate;
    int groups, B, H, W, C, Hp, Wp, Pp, halo;
    int tiles_m, tiles_n, total_tiles, chunk;
    int units;               // FWD, DX: parts of 64 padded pixels per group (pool_part, stat_part)
    int strip_pieces, strip_bytes;   // FWD, DX: the strip in pieces of eight rows; its (or the staging's) place in LDS
    FastDiv div_per, div_wp; // division by (H + 2) (W + 2) and by W + 2
    FastDiv div_pg, div_tn;  // FWD, DX: division by tiles_m * tiles_n and by tiles_n
    int splits, k_chunk;
};

__device__ __forceinline__ int xcd_tile(int chunk, int total) {
    const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
    const int tile = xcd * chunk + slot;
    return (slot >= chunk || tile >= total) ? -1 : tile;
}

// padded pixel q -> is it an image pixel, and which (index in the unpadded [B H W] order)
__device__ __forceinline__ bool interior(const ConvBDev& p, int q, int* unpadded) {
    const int per = p.Hp * p.Wp;
    const int n = (int)fast_div((unsigned)q, p.div_per), rem = q - n * per;
    const int y = (int)fast_div((unsigned)rem, p.div_wp), x = rem - y * p.Wp;
    *unpadded = (n * p.H + (y - 1)) * p.W + (x - 1);
    return y >= 1 && y <= p.H && x >= 1 && x <= p.W;
}

// Two sign bytes of eight bf16 channels that are not negative (a ReLU's result): bit e of byte b is set iff channel 4 b + e is
// positive.  The magnitude's 15 bits plus 0x7FFF carry into bit 15 unless they are all zero; the eight carries then close up.
__device__ __forceinline__ unsigned short positive_bits(u4 v) {
    u4 c;
#pragma unroll
    for (int w = 0; w < 4; ++w) c[w] = ((v[w] & 0x7FFF7FFFu) + 0x7FFF7FFFu) & 0x80008000u;
    const unsigned u = c[0] >> 15 | c[1] >> 13 | c[2] >> 7 | c[3] >> 5;   // channels 0, 2, 4, 6 at 0, 2, 8, 10; their successors 16 above
    return (unsigned short)((u | u >> 15) & 0x0F0Fu);
}

// ---------------------------------------------------------------------------------------------
// forward (MODE 0) and back-propagated delta (MODE 1)
// ---------------------------------------------------------------------------------------------
// What the epilogue produces: bf16 in the padded operand layout; conv + bias in fp32, padded; the fused tail; or fp32 in
// the UNPADDED [B H W][C] layout (image pixels only) -- the input of a batch normalisation (forward) or of its backward
// pass (delta, gated by the sign of the bf16 activation as usual).
enum { kOutBf16 = 0, kOutF32 = 1, kOutTail = 2, kOutF32U = 3 };
constexpr int kHalfRows = 64;             // rows that a wavefront's epilogue stages and moves at a time
constexpr int kStripRow = 2 * kCB;        // bytes of a strip row (one pixel's 64 channels)
__host__ __device__ constexpr int stage_pitch(int out, int bn) { return out == kOutBf16 ? 2 * (bn + 8) : 4 * (bn + 4); }   // bytes
__host__ __device__ constexpr int stage_bytes(int out, int bn) { return 4 * kHalfRows * stage_pitch(out, bn); }            // of the four wavefronts
constexpr bool row_index(int out) { return out == kOutTail || out == kOutF32U; }   // the epilogue needs the rows' unpadded pixel indices

// A workgroup's tile is 128 TM padded pixels x 32 TN output channels; a wavefront owns 32 TM pixels x 32 TN channels.
// LDS: the strip (later the epilogue's staging), a table of the tile's rows, the bias.
template <int MODE, int OUT, int TM, int TN>
__global__ __launch_bounds__(kThreads, 2) void conv3x3_bf16_kernel(ConvBDev p) {
    constexpr int BM = 128 * TM, WR = 32 * TM, BN = 32 * TN;
    constexpr int KS = kCB / 16, kSteps = 9 * KS;       // contraction steps of a chunk: (tap, 16 channels)
    constexpr int kAhead = 4;                           // kernel fragments are requested that many steps ahead
    static_assert(WR % kHalfRows == 0, "the epilogue works on whole halves");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    int* row_up = (int*)(lds + p.strip_bytes);          // [BM] image pixel: its index in the unpadded [B H W] order; border: -1
    float* bias_lds = (float*)(row_up + BM);            // [BN]

    const int tile = xcd_tile(p.chunk, p.total_tiles);
    if (tile < 0) return;
    OLS_TP(0);   // first instruction after the tile is known
    const int per_group = p.tiles_m * p.tiles_n;
    const int group = (int)fast_div((unsigned)tile, p.div_pg);
    const int in_group = tile - group * per_group;
    const int tm = (int)fast_div((unsigned)in_group, p.div_tn), tn = in_group - tm * p.tiles_n;
    const int m0 = tm * BM, n0 = tn * BN;
    const int C = p.C, nb = C / kCB;

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const int lane32 = lane % 32, half = lane / 32;
    const int wm0 = wave * WR;

    const unsigned row_bytes = 2u * (unsigned)C;
    const rsrc_t in_rs = make_rsrc(p.in + (int64_t)group * p.s_in, (unsigned)p.Pp * row_bytes);
    const rsrc_t w_rs = make_rsrc(p.w + (int64_t)group * p.s_w, 9u * (unsigned)C * row_bytes);
    // Rows m0 - halo .. of channels c0 .. c0 + 63, loaded straight into LDS: a wavefront's instruction fills eight rows
    // (1 KiB, lane by lane), and a lane fetches the 16-byte vector that belongs at its place -- vector v of row r lies at
    // place v ^ (r % 8), so that eight lanes reading one vector of eight consecutive rows cover all banks.  Rows before the
    // tensor wrap to offsets beyond its end, rows after it lie beyond it too: both arrive as zeros.
    const unsigned strip_lane = (unsigned)(m0 - p.halo + lane / 8) * row_bytes + ((lane % 8) ^ (lane / 8)) * 16u;
    auto load_strip = [&](int c0) {
        for (int t = wave; t < p.strip_pieces; t += 4)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(in_rs, (lds_void_ptr)(lds + t * 1024), 16, (int)(strip_lane + t * 8u * row_bytes), 2 * c0, 0, 0);
    };
    // Fragments of the kernels come in their own order (see kernel_images) straight into registers: no LDS, no barrier
    // between the taps.  The last chunk's requests past its end lie outside the range and cost nothing.
    bf16x8 fa[2][TM], fb[kAhead][TN];
    const int jn = (n0 / 32) % 2;
    auto load_fb = [&](int slot, int k, int c) {
        const unsigned first = (unsigned)(((k / KS) * nb + c) * nb + n0 / kCB) * (kCB * kCB * 2u) + (2 * (k % KS) + jn) * 1024u;
        const unsigned off = c < nb ? lane * 16u : 0x40000000u;
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[slot][j] = __builtin_bit_cast(bf16x8, buf_load(w_rs, off, first + j * 1024u));
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
    int fa_row = 0;
    auto load_fa = [&](int buf, int k) {
        const int tap = k / KS, s = k % KS;
        int row = wm0 + lane32 + p.halo + (MODE == 0 ? 1 : -1) * ((tap / 3 - 1) * p.Wp + tap % 3 - 1);
        if (s == 0) asm("" : "+v"(row));   // (or the compiler keeps the addresses of all steps across the chunks: 40 registers)
        else row = fa_row;
        fa_row = row;
        const uint8_t* a = lds + row * kStripRow + ((half ^ (row & 7) ^ (2 * s)) * 16);
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[buf][i] = __builtin_bit_cast(bf16x8, *(const u4*)(a + i * 32 * kStripRow));
    };

    // What the epilogue reads from memory is requested two taps before the end: delta, the sign bytes that gate the result, a row
    // of the wavefront per lane; fused tail, the shortcut's fp32 rows in batches of eight vectors per lane, the first then and
    // each further one while the batch before it is consumed.
    constexpr int kVecB = BN / 8, kVecF = BN / 4;       // vectors of a row: bf16 and fp32
    constexpr int kRowsB = 64 / kVecB, kRowsF = 64 / kVecF;   // rows that a wavefront moves at a time
    constexpr int kHalves = WR / kHalfRows, kTailBatch = TM == 4 ? 8 : 4, kBatches = kVecF / kTailBatch;
    typedef typename std::conditional<TN == 2, u4, u2>::type gate_row;   // a row's sign bytes: BN / 4 of them
    gate_row gates[MODE == 1 ? kHalves : 1];
    const unsigned own_b = (unsigned)(m0 + wm0 + lane / kVecB) * row_bytes + 2u * (unsigned)n0 + (lane % kVecB) * 16u;
    auto load_gates = [&]() {
        const unsigned rows = OUT == kOutF32U ? (unsigned)(p.B * p.H * p.W) : (unsigned)p.Pp;   // of the output, like the bytes
        const rsrc_t rs = make_rsrc(p.gate + (int64_t)group * p.s_gate, rows * (unsigned)(C / 4));
#pragma unroll
        for (int h = 0; h < kHalves; ++h) {
            const int r = wm0 + h * kHalfRows + lane;
            const unsigned off = (unsigned)(OUT == kOutF32U ? row_up[r] : m0 + r) * (unsigned)(C / 4) + n0 / 4;   // border rows: -1, beyond the range
            if constexpr (TN == 2) gates[h] = buf_load(rs, off, 0u);
            else gates[h] = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)off, 0, 0);
        }
    };
    f4 xres[OUT == kOutTail ? kTailBatch : 1];
    int up_res[OUT == kOutTail ? kTailBatch : 1];
    const rsrc_t x_rs = make_rsrc(OUT == kOutTail ? (const void*)(p.xres + (int64_t)group * p.s_x) : (const void*)p.in,
                                  OUT == kOutTail ? (unsigned)(p.B * p.H * p.W) * 2u * row_bytes : 0u);
    auto load_shortcut = [&](int batch) {   // batch counts over both halves
#pragma unroll
        for (int t = 0; t < kTailBatch; ++t) up_res[t] = row_up[wm0 + lane / kVecF + kRowsF * (kTailBatch * batch + t)];
#pragma unroll
        for (int t = 0; t < kTailBatch; ++t)   // border rows: -1 wraps to an offset beyond the tensor, zeros come back
            xres[t] = __builtin_bit_cast(f4, buf_load(x_rs, (unsigned)up_res[t] * 2u * row_bytes + 4u * n0 + (lane % kVecF) * 16u, 0u));
    };

    for (int c = 0; c < nb; ++c) {
        // the previous chunk's last barrier has passed: nobody reads the strip any more
        load_strip(kCB * c);
        if (c == 0) {
#pragma unroll
            for (int k = 0; k < kAhead; ++k) load_fb(k, k, 0);
            OLS_TP(1);   // the chunk's loads are issued
#pragma unroll
            for (int r = threadIdx.x; r < BM; r += kThreads) {   // which rows of the tile are image pixels
                int up;
                row_up[r] = m0 + r < p.Pp && interior(p, m0 + r, &up) ? up : -1;
            }
            if (MODE == 0 && threadIdx.x < BN) bias_lds[threadIdx.x] = p.bias ? p.bias[(int64_t)group * p.s_bias + n0 + threadIdx.x] : 0.0f;
        }
        // Loads into LDS count as vector loads, and the barrier alone waits for no wavefront's: each waits for its own rows first
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        OLS_TP(2);   // the strip is in LDS
        load_fa(0, 0);
#pragma unroll
        for (int k = 0; k < kSteps; ++k) {
            if (k == 7 * KS) {   // in every chunk: a branch here would make the waits on the fragments wait for these too
                if constexpr (MODE == 1) load_gates();
                if constexpr (OUT == kOutTail) load_shortcut(0);
            }
            if (k + 1 < kSteps) load_fa((k + 1) & 1, k + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[k % kAhead][j], fa[k & 1][i], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            load_fb(k % kAhead, (k + kAhead) % kSteps, k + kAhead < kSteps ? c : c + 1);
        }
        __syncthreads();
    }
    static_assert(kSteps % kAhead == 0, "a chunk's first fragments lie in the first slots");

    OLS_TP(3);   // the taps are done
    // Epilogue: the tile goes through LDS (the strip's place) so that every lane then moves 16-byte vectors.  A wavefront
    // stages and moves its own rows, 64 at a time: its LDS operations complete in order, so no workgroup barrier is needed
    // after the one that ended the last tap.
    constexpr int kPitch = stage_pitch(OUT, BN);
    uint8_t* stage = lds + wave * kHalfRows * kPitch;
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    auto put = [&](int h, auto store) {   // hands the half's accumulators out as quads (row, channel, values)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    const f16v& t = acc[2 * h + i][j];
                    f4 o = {t[4 * g4], t[4 * g4 + 1], t[4 * g4 + 2], t[4 * g4 + 3]};
                    const int n = 32 * j + 8 * g4 + 4 * half;
                    if constexpr (MODE == 0 && OUT != kOutF32U) o = o + *(const f4*)(bias_lds + n);
                    store(32 * i + lane32, n, o);
                }
    };
    // Sign bytes of the half's rows, behind the staging areas: they cross memory a row per lane and are used, or made, where
    // the lanes hold vectors (stored from there, 16 or 32 stores of a byte or two per lane, they cost the forward kernel 23 us)
    uint8_t* gate_lds = lds + stage_bytes(OUT, BN) + wave * (kHalfRows * BN / 4);
    auto store_gates = [&](rsrc_t rs, int h) {
        const unsigned off = (unsigned)(m0 + wm0 + h * kHalfRows + lane) * (unsigned)(C / 4) + n0 / 4;   // rows past the tensor are dropped
        const gate_row v = *(const gate_row*)(gate_lds + lane * (BN / 4));
        if constexpr (TN == 2) buf_store(v, rs, off);
        else __builtin_amdgcn_raw_buffer_store_b64(v, rs, (int)off, 0, 0);
    };
    auto put_gates = [&](int h) {
        if constexpr (MODE == 1) *(gate_row*)(gate_lds + lane * (BN / 4)) = gates[h];
    };
    auto put_f32 = [&](int r, int n, f4 o) { *(f4*)(stage + r * kPitch + 4 * n) = o; };
    const int r0 = lane / kVecF, cq = lane % kVecF;     // fp32 staging: lane owns the channel quad cq of rows r0 + kRowsF t
    auto staged = [&](int t) { return *(const f4*)(stage + (r0 + kRowsF * t) * kPitch + cq * 16); };
    // sum over the kRowsF lanes of a channel quad, in lane order, through 64 vectors of LDS that no lane needs any more
    auto quad_sum = [&](f4* red, f4 v, int q) {
        red[lane] = v;
        wave_sync();
        f4 o = red[q];
#pragma unroll
        for (int u = 1; u < kRowsF; ++u) o = o + red[u * kVecF + q];
        return o;
    };

    if constexpr (OUT == kOutTail) {
        // a2 = relu(convolution + bias + shortcut) on the image pixels: its sign bytes and, per 64 consecutive padded pixels
        // (which touch at most two samples because a padded image has at least 64), the channel sums of its rows in the
        // first and in the second of those samples.  A later pass adds these sums per sample in order.
        const rsrc_t sg_rs = make_rsrc(p.sign + (int64_t)group * p.s_sign, (unsigned)p.Pp * (unsigned)(C / 4));
        const int per = p.Hp * p.Wp;
#pragma unroll
        for (int h = 0; h < kHalves; ++h) {
            const int q0 = m0 + wm0 + h * kHalfRows;                    // the half's first padded pixel
            const int next_sample = ((int)fast_div((unsigned)q0, p.div_per) + 1) * per;   // first pixel of the second sample
            put(h, put_f32);
            wave_sync();
            f4 sum0 = {0.f, 0.f, 0.f, 0.f}, sum1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int b = 0; b < kBatches; ++b) {
                f4 yv[kTailBatch], xv[kTailBatch];
                int up[kTailBatch];
#pragma unroll
                for (int t = 0; t < kTailBatch; ++t) { up[t] = up_res[t]; xv[t] = xres[t]; }
                if (h * kBatches + b + 1 < kHalves * kBatches) load_shortcut(h * kBatches + b + 1);   // travels while this one is consumed
#pragma unroll
                for (int t = 0; t < kTailBatch; ++t) yv[t] = staged(kTailBatch * b + t);
#pragma unroll
                for (int t = 0; t < kTailBatch; ++t) {
                    const int q = q0 + r0 + kRowsF * (kTailBatch * b + t);
                    const bool img = up[t] >= 0;
                    unsigned bits = 0;
                    f4 a;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        a[e] = img ? fmaxf(yv[t][e] + xv[t][e], 0.0f) : 0.0f;
                        bits |= a[e] > 0.0f ? (1u << e) : 0u;
                    }
                    if (q < next_sample) sum0 = sum0 + a; else sum1 = sum1 + a;
                    gate_lds[(r0 + kRowsF * (kTailBatch * b + t)) * (BN / 4) + cq] = (uint8_t)bits;
                }
            }
            wave_sync();   // all reads of the staging area are done
            store_gates(sg_rs, h);
            const int unit = tm * (BM / kHalfRows) + wave * kHalves + h;
            const f4 o0 = quad_sum((f4*)stage, sum0, cq), o1 = quad_sum((f4*)stage + 64, sum1, cq);
            if (lane < kVecF && unit < p.units) {
                float* PP = p.pool_part + ((int64_t)group * p.units + unit) * 2 * C + n0 + 4 * cq;
                *(f4*)PP = o0;
                *(f4*)(PP + C) = o1;
            }
            wave_sync();
        }
    } else if constexpr (OUT == kOutF32 || OUT == kOutF32U) {
        // Convolution + bias only (what follows it is another kernel's).  Padded output: border rows are written as
        // computed; their consumer skips them.  Unpadded output: a row goes to its pixel's place in the [B H W] order and a
        // border row to offset -1, which the range check drops.
        const unsigned out_rows = OUT == kOutF32U ? (unsigned)(p.B * p.H * p.W) : (unsigned)p.Pp;
        const rsrc_t out_rs = make_rsrc((const float*)p.out + (int64_t)group * p.s_out, out_rows * 2u * row_bytes);
        const unsigned col_off = 4u * (unsigned)n0 + cq * 16u;
#pragma unroll
        for (int h = 0; h < kHalves; ++h) {
            const int hr = wm0 + h * kHalfRows;
            put_gates(h);
            put(h, put_f32);
            wave_sync();
            f4 zv[kVecF];
            int up[kVecF], bits[MODE == 1 ? kVecF : 1];
#pragma unroll
            for (int t = 0; t < kVecF; ++t) {
                zv[t] = staged(t);
                up[t] = row_up[hr + r0 + kRowsF * t];
                if constexpr (MODE == 1) bits[t] = gate_lds[(r0 + kRowsF * t) * (BN / 4) + cq];
            }
#pragma unroll
            for (int t = 0; t < kVecF; ++t) {
                u4 o = __builtin_bit_cast(u4, zv[t]);
                if constexpr (MODE == 1) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = ((unsigned)bits[t] >> e) & 1u ? o[e] : 0u;
                }
                if constexpr (OUT == kOutF32U) buf_store(o, out_rs, (unsigned)up[t] * 2u * row_bytes + col_off);   // border rows: dropped
                else buf_store(o, out_rs, (unsigned)(m0 + hr + r0 + kRowsF * t) * 2u * row_bytes + col_off);        // rows past the tensor are dropped
            }
            wave_sync();
            if constexpr (MODE == 0 && OUT == kOutF32U) {
                // Statistics of these 64 padded pixels' image pixels for the batch normalisation that follows (which then
                // need not read the output again): count, mean, and the sum of squared deviations from that mean, per
                // channel.  A later pass merges the parts in order (the parallel-variance rule).
                if (p.stat_part) {
                    f4* red = (f4*)stage;
                    f4 sum = {0.f, 0.f, 0.f, 0.f};
                    float cnt = 0.0f;
#pragma unroll
                    for (int t = 0; t < kVecF; ++t)
                        if (up[t] >= 0) { sum = sum + zv[t]; cnt += 1.0f; }
                    const f4 tot = quad_sum(red, sum, cq);
                    float n = __shfl(cnt, cq);
#pragma unroll
                    for (int u = 1; u < kRowsF; ++u) n += __shfl(cnt, u * kVecF + cq);
                    const float inv_n = n > 0.0f ? 1.0f / n : 0.0f;
                    f4 mean;
#pragma unroll
                    for (int e = 0; e < 4; ++e) mean[e] = tot[e] * inv_n;
                    f4 dev = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int t = 0; t < kVecF; ++t)
                        if (up[t] >= 0) { const f4 d = zv[t] - mean; dev = dev + d * d; }
                    const f4 m2 = quad_sum(red + 64, dev, cq);
                    const int unit = tm * (BM / kHalfRows) + wave * kHalves + h;
                    if (lane < kVecF && unit < p.units) {
                        float* SP3 = p.stat_part + ((int64_t)group * p.units + unit) * 3 * C + n0 + 4 * cq;
                        *(f4*)SP3 = f4{n, n, n, n};
                        *(f4*)(SP3 + C) = mean;
                        *(f4*)(SP3 + 2 * C) = m2;
                    }
                    wave_sync();
                }
            }
        }
    } else {
        const rsrc_t out_rs = make_rsrc((const uint16_t*)p.out + (int64_t)group * p.s_out, (unsigned)p.Pp * row_bytes);
        const rsrc_t gate_rs = make_rsrc(p.gate + (int64_t)group * p.s_gate, (unsigned)p.Pp * (unsigned)(C / 4));
#pragma unroll
        for (int h = 0; h < kHalves; ++h) {
            put_gates(h);
            put(h, [&](int r, int n, f4 v) {
                if constexpr (MODE == 0) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.0f);   // ReLU
                }
                u2 o;   // round to nearest even (v_cvt_pk_bf16_f32)
                o.x = __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{v[0], v[1]}, bf16x2));
                o.y = __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{v[2], v[3]}, bf16x2));
                *(u2*)(stage + r * kPitch + 2 * n) = o;
            });
            wave_sync();
            u4 val[kVecB];
            int flag[kVecB];   // FWD: < 0 in the border; DX: the two sign bytes
#pragma unroll
            for (int t = 0; t < kVecB; ++t) {
                const int r = lane / kVecB + kRowsB * t;
                val[t] = *(const u4*)(stage + r * kPitch + (lane % kVecB) * 16);
                flag[t] = MODE == 0 ? row_up[wm0 + h * kHalfRows + r] : *(const uint16_t*)(gate_lds + r * (BN / 4) + lane % kVecB * 2);
            }
#pragma unroll
            for (int t = 0; t < kVecB; ++t) {
                u4 o = val[t];
                if constexpr (MODE == 0) {
                    if (flag[t] < 0) o = u4{0u, 0u, 0u, 0u};   // the zero border the next layer relies on
                    *(unsigned short*)(gate_lds + (lane / kVecB + kRowsB * t) * (BN / 4) + lane % kVecB * 2) = positive_bits(o);
                } else {
                    const unsigned bits = flag[t];
#pragma unroll
                    for (int w = 0; w < 4; ++w) {   // channels 2 w and 2 w + 1: bits 2 w, 2 w + 1 of their byte
                        const unsigned two = bits >> (w < 2 ? 2 * w : 8 + 2 * (w - 2));
                        o[w] &= (two & 1u ? 0xFFFFu : 0u) | (two & 2u ? 0xFFFF0000u : 0u);
                    }
                }
                buf_store(o, out_rs, own_b + (h * kHalfRows + t * kRowsB) * row_bytes);   // rows past the tensor are dropped
            }
            wave_sync();
            if constexpr (MODE == 0) store_gates(gate_rs, h);
        }
    }
    OLS_TP(4);   // the tile's stores are issued
}

// ---------------------------------------------------------------------------------------------
// kernel / bias gradient.  One workgroup per (pixel range, 64 x 64 block of input x output channels): twelve wavefronts
// (three per SIMD), (kernel row, 32 input channels, half of the contraction steps) each, with 32 x 64 channels x three taps in
// 96 accumulators per lane; the halves are added through LDS at the end.  96 padded pixels per slice; the input rows live in
// a ring of 512 LDS rows, so each is fetched once
// although nine taps read it at nine offsets, and the delta's rows alternate between two buffers.  Rows are 128 bytes, their
// halves exchanged by bit 1 of the row, so that the four rows of a transpose read cover the 64 banks.  A lane's fragments of
// the three taps are eight of the pixels -1 .. 8 around its own eight: three transpose reads bring -1 .. 10 (the last two are
// not used, and may be rows that are being written).
// ---------------------------------------------------------------------------------------------
constexpr int kDwThreads = 768, kDwRing = 512, kDwRow = 128, kDwVecs = 2;   // LDS rows in bytes; vectors per copying lane
static_assert(kDwBK * 8 == kDwVecs * kDwThreads / 2, "half of the lanes copy input rows, half the delta's");
constexpr int kDwFold = 6 * 64 * 96 * 4;   // bytes of one half's accumulators, which take the operands' place in LDS
static_assert((kDwRing + 2 * kDwBK) * kDwRow <= kDwFold, "the larger of the two");
static_assert(2 * kDwBK + 2 * (kConvBf16MaxWidth + 3) <= kDwRing, "the ring holds a slice's window and the next slice's rows");
__global__ __launch_bounds__(kDwThreads, 3) void conv3x3_dw_bf16_kernel(ConvBDev p) {
    extern __shared__ __attribute__((aligned(16))) uint8_t dw_lds[];
    uint8_t* ring = dw_lds;
    auto delta = [&](int buf) { return dw_lds + kDwRing * kDwRow + buf * (kDwBK * kDwRow); };

    const int tile = xcd_tile(p.chunk, p.total_tiles);
    if (tile < 0) return;
    const int nb = p.tiles_n;                                    // 64-channel blocks
    const int per_group = p.splits * nb * nb;
    const bool second = tile >= p.layer_tiles;
    const int in_layer = second ? tile - p.layer_tiles : tile;
    const int group = in_layer / per_group;
    const int rest = in_layer % per_group;
    const int split = rest / (nb * nb);
    const int ci0 = ((rest / nb) % nb) * kCB, co0 = (rest % nb) * kCB;
    const int lo = split * p.k_chunk, hi = min(p.Pp, lo + p.k_chunk);
    const int C = p.C;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const int kh = wave / 4, wi = (wave / 2) % 2, khalf = wave % 2;

    // Copying: lanes 0 .. 383 move input rows, 384 .. 767 delta rows; vector t % 8 of rows t / 8 and t / 8 + 48.  Input rows
    // outside the tensor read as zeros, and so do the delta's rows from the end of the range on (its descriptor ends there).
    const bool moves_in = wave < kDwThreads / 128;   // (in scalar registers, like the descriptor)
    const int mt = moves_in ? threadIdx.x : threadIdx.x - kDwThreads / 2;
    const int mrow = mt / 8, mv = mt % 8;
    const unsigned row_bytes = 2u * (unsigned)C;
    const uint16_t* src = moves_in ? (second ? p.in_b : p.in) + (int64_t)group * p.s_in : (second ? p.dout_b : p.dout) + (int64_t)group * p.s_dout;
    const rsrc_t rs = make_rsrc(src, (unsigned)(moves_in ? p.Pp : hi) * row_bytes);
    const unsigned lane_off = 2u * (unsigned)(moves_in ? ci0 : co0) + mv * 16u;
    auto load_rows = [&](u4 (&r)[kDwVecs], int q0) {   // (a negative row wraps to an offset beyond the range)
#pragma unroll
        for (int t = 0; t < kDwVecs; ++t) r[t] = buf_load(rs, (unsigned)(q0 + mrow + 48 * t) * row_bytes + lane_off, 0u);
    };
    // bias gradient: the delta's column sums, from the fragments of the first kernel row's wavefronts (a lane holds eight
    // pixels of one channel)
    const bool col_sums = ci0 == 0;
    float col_acc[2] = {0.0f, 0.0f};
    uint8_t* put_base = moves_in ? ring : delta(0);
    auto put_rows = [&](const u4 (&r)[kDwVecs], int row0) {
#pragma unroll
        for (int t = 0; t < kDwVecs; ++t) {
            const int row = (row0 + mrow + 48 * t) & (kDwRing - 1);
            *(u4*)(put_base + row * kDwRow + (((mv / 4) ^ ((row >> 1) & 1)) * 64) + (mv % 4) * 16) = r[t];
        }
    };

    const int blk = lane / 16, j = lane % 16;
    const int frow = 8 * (blk / 2) + j / 4, fcol = (16 * (blk % 2) + 4 * (j % 4)) * 2;
    typedef s4v __attribute__((address_space(3))) * lds_s4_ptr;
    auto row_addr = [&](int row, int piece) { return row * kDwRow + ((piece ^ ((row >> 1) & 1)) * 64) + fcol; };
    auto quad = [&](const uint8_t* a) { return __builtin_bit_cast(u2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)a)); };   // four pixels of a lane's channel
    f16v acc[3][2];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[t][c][e] = 0.0f;

    // ring row of padded pixel q: (q - lo + halo) mod 512
    const int nslices = hi > lo ? (hi - lo + kDwBK - 1) / kDwBK : 0;
    if (nslices > 0) {
        u4 r0[kDwVecs], r1[kDwVecs];
        const int ahead = moves_in ? p.halo : 0;
        if (moves_in) {
            for (int d = 0; d < kDwBK + 2 * p.halo; d += kDwBK) {
                load_rows(r0, lo - p.halo + d);
                put_rows(r0, d);
            }
        } else {
            load_rows(r0, lo);
            put_rows(r0, 0);
        }
        load_rows(r0, lo + kDwBK + ahead);
        __syncthreads();
        auto slice = [&](int t, const u4 (&next)[kDwVecs], u4 (&after)[kDwVecs]) {
            load_rows(after, lo + (t + 2) * kDwBK + ahead);       // (past the range: zeros that nothing reads)
            __builtin_amdgcn_sched_barrier(0);
            const uint8_t* D = delta(t & 1);
            const int base = t * kDwBK + p.halo + (kh - 1) * p.Wp + frow;
#pragma unroll
            for (int s = 0; s < kDwBK / 32; ++s) {                // of this wavefront's half
                const int k16 = 16 * (2 * s + khalf);
                bf16x8 fd[2];
                u2 w[3];                                          // input pixels -1 .. 10 of a lane's eight: the three taps
#pragma unroll
                for (int q = 0; q < 3; ++q) w[q] = quad(ring + row_addr((base + k16 - 1 + 4 * q) & (kDwRing - 1), wi));
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const uint8_t* a = D + row_addr(k16 + frow, c);
                    fd[c] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(quad(a), quad(a + 4 * kDwRow), 0, 1, 2, 3));   // four rows on: the same bit 1
                }
                const unsigned px[5] = {w[0].x, w[0].y, w[1].x, w[1].y, w[2].x};
#pragma unroll
                for (int kw = 0; kw < 3; ++kw) {
                    u4 f;
#pragma unroll
                    for (int e = 0; e < 4; ++e) f[e] = kw == 0 ? px[e] : kw == 1 ? __builtin_amdgcn_alignbit(px[e + 1], px[e], 16) : px[e + 1];
#pragma unroll
                    for (int c = 0; c < 2; ++c) acc[kw][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f), fd[c], acc[kw][c], 0, 0, 0);
                }
                if (col_sums && kh == 0 && wi == 0) {
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const u4 d = __builtin_bit_cast(u4, fd[c]);
#pragma unroll
                        for (int e = 0; e < 4; ++e) col_acc[c] += __uint_as_float(d[e] << 16) + __uint_as_float(d[e] & 0xFFFF0000u);
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            put_rows(next, moves_in ? (t + 1) * kDwBK + 2 * p.halo : ((t + 1) & 1) * kDwBK);   // behind the window; the other buffer
            __syncthreads();
        };
        int t = 0;
        for (; t + 1 < nslices; t += 2) {
            slice(t, r0, r1);
            slice(t + 1, r1, r0);
        }
        if (t < nslices) slice(t, r0, r1);
    }

    // the second half of the steps hands its sums over (the operand rows are no longer read)
    float* fold = (float*)dw_lds + (wave / 2) * (64 * 96) + lane;
    if (khalf == 1) {
#pragma unroll
        for (int kw = 0; kw < 3; ++kw)
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int e = 0; e < 16; ++e) fold[((2 * kw + c) * 16 + e) * 64] = acc[kw][c][e];
    }
    __syncthreads();
    const int64_t n_w = (int64_t)9 * C * C;
    float* PART = (second ? p.partial_b : p.partial) + ((int64_t)split * p.groups + group) * (n_w + C);
    if (khalf == 0) {
#pragma unroll
        for (int kw = 0; kw < 3; ++kw)
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int ci = ci0 + 32 * wi + 8 * (e / 4) + 4 * (lane / 32) + (e % 4);
                    PART[((int64_t)(3 * kh + kw) * C + ci) * C + co0 + 32 * c + lane % 32] = acc[kw][c][e] + fold[((2 * kw + c) * 16 + e) * 64];
                }
    }
    if (ci0 == 0) {   // channel c: the two halves of the steps, both halves of the wavefronts' lanes, added in a fixed order
        __syncthreads();
        float* red = (float*)dw_lds;
        if (kh == 0 && wi == 0) {
            red[khalf * 128 + lane] = col_acc[0];
            red[khalf * 128 + 64 + lane] = col_acc[1];
        }
        __syncthreads();
        if (threadIdx.x < kCB) {
            const float* r = red + 64 * (threadIdx.x / 32) + threadIdx.x % 32;
            PART[n_w + co0 + threadIdx.x] = ((r[0] + r[32]) + r[128]) + r[160];
        }
    }
}

// ---------------------------------------------------------------------------------------------
// fp32 [B H W][C] -> bf16 [B (H+2) (W+2)][C] with a zero border; one lane per 8 channels of a padded pixel
// ---------------------------------------------------------------------------------------------
// The kernels of a step in the order in which the forward / delta kernel's lanes take their fragments: one 64 x 64 slice per
// (tap, 64-channel chunk of the contraction, 64 output channels), in it [step of 16][32 output channels][lane][8]: lane l holds
// contraction channels 16 s + 8 (l / 32) .. + 7 of output channel 32 j + l % 32.  Three images: the first convolution's
// kernels, the second's, and the second's with its channel indices exchanged (for the delta).  One workgroup per slice.
struct KernelImages {
    const uint16_t* w[3];    // [9][C][C] per group
    uint16_t* dst[3];        // [9 C C] per group
    int64_t s_w, s_dst;
    int C;
};
__device__ __forceinline__ void kernel_images(const KernelImages& im, int unit, int group) {
    const int nb = im.C / kCB, which = unit / (9 * nb * nb), slice = unit % (9 * nb * nb);
    const int tap = slice / (nb * nb), c0 = (slice / nb % nb) * kCB, n0 = (slice % nb) * kCB;
    const uint16_t* W = im.w[which] + (int64_t)group * im.s_w + (int64_t)tap * im.C * im.C;
    u4* D = (u4*)(im.dst[which] + (int64_t)group * im.s_dst + (int64_t)slice * (kCB * kCB));
#pragma unroll
    for (int v = threadIdx.x; v < kCB * kCB / 8; v += kThreads) {
        const int l = v % 64, n = n0 + 32 * (v / 64 % 2) + l % 32, k = c0 + 16 * (v / 128) + 8 * (l / 32);
        u4 o;
        if (which == 2) {
            o = *(const u4*)(W + (int64_t)n * im.C + k);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                o[e] = W[(int64_t)(k + 2 * e) * im.C + n] | (unsigned)W[(int64_t)(k + 2 * e + 1) * im.C + n] << 16;
        }
        D[v] = o;
    }
}

constexpr int kPadCastFly = 2;   // 16-byte output vectors per lane
template <bool STREAM>   // non-temporal loads of the batch (tensors_stream)
__global__ __launch_bounds__(kThreads) void pad_cast_bf16_kernel(const float* __restrict__ src, int64_t s_src,
                                                                 uint16_t* __restrict__ dst, int64_t s_dst, unsigned vecs, int H,
                                                                 int W, int C, FastDiv div_c8, FastDiv div_per, FastDiv div_wp,
                                                                 KernelImages im, unsigned image_blocks) {
    const int g = blockIdx.y;
    if (blockIdx.x < image_blocks) {   // the step's kernels travel with its batch
        kernel_images(im, blockIdx.x, g);
        return;
    }
    const unsigned block = blockIdx.x - image_blocks;
    const unsigned c8 = (unsigned)C / 8, Wp = (unsigned)W + 2, per = (unsigned)(H + 2) * Wp;
    f4 lo[kPadCastFly], hi[kPadCastFly];
    bool img[kPadCastFly];
#pragma unroll
    for (int t = 0; t < kPadCastFly; ++t) {   // the loads of all the lane's vectors before the first store
        const unsigned v = (block * kPadCastFly + t) * kThreads + threadIdx.x;
        const unsigned q = fast_div(v < vecs ? v : 0u, div_c8), cv = (v < vecs ? v : 0u) - q * c8;
        const unsigned n = fast_div(q, div_per), rem = q - n * per;
        const unsigned y = fast_div(rem, div_wp), x = rem - y * Wp;
        img[t] = v < vecs && y >= 1 && y <= (unsigned)H && x >= 1 && x <= (unsigned)W;
        if (img[t]) {
            const f4* S = (const f4*)(src + (int64_t)g * s_src + ((int64_t)(n * H + y - 1) * W + (x - 1)) * C) + 2 * cv;
            lo[t] = STREAM ? __builtin_nontemporal_load(S) : S[0];
            hi[t] = STREAM ? __builtin_nontemporal_load(S + 1) : S[1];
        }
    }
#pragma unroll
    for (int t = 0; t < kPadCastFly; ++t) {
        const unsigned v = (block * kPadCastFly + t) * kThreads + threadIdx.x;
        if (v >= vecs) continue;
        u4 o = {0u, 0u, 0u, 0u};
        if (img[t]) {   // round to nearest even (v_cvt_pk_bf16_f32)
            o.x = __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{lo[t][0], lo[t][1]}, bf16x2));
            o.y = __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{lo[t][2], lo[t][3]}, bf16x2));
            o.z = __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{hi[t][0], hi[t][1]}, bf16x2));
            o.w = __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{hi[t][2], hi[t][3]}, bf16x2));
        }
        *((u4*)(dst + (int64_t)g * s_dst) + v) = o;
    }
}

// The block's tail in one streaming pass: a2 = relu(y + X) for the image pixels of one (sample, worker), its mean over
// the positions (global average pooling), and the sign of a2 for the backward pass -- a2 itself is needed nowhere else,
// so it is never written.  y: convolution output + bias, fp32 [Pp][C] with border rows (skipped); X: the shortcut, fp32
// [B H W][C]; sign[q][c / 4]: one byte per padded pixel and four channels, bit e set iff a2[q][4 (c / 4) + e] > 0 (border: 0).
// One workgroup per (sample, worker); thread = (channel vector, position stripe); stripes combined in a fixed order.
__global__ __launch_bounds__(kThreads) void shortcut_relu_pool_kernel(const float* __restrict__ y, int64_t s_y,
                                                                      const float* __restrict__ X, int64_t s_x, float* pooled,
                                                                      int64_t s_p, uint8_t* sign, int64_t s_sign, int H, int W, int C,
                                                                      FastDiv div_wp, float inv) {
    __shared__ f4 part[kThreads];
    const int c4n = C / 4, stripes = kThreads / c4n;
    const int c4 = threadIdx.x % c4n, stripe = threadIdx.x / c4n;
    const int b = blockIdx.x, g = blockIdx.y;
    const int Wp = W + 2, per = (H + 2) * Wp;
    const float* Y = y + (int64_t)g * s_y + (int64_t)b * per * C + 4 * c4;
    const float* Xs = X + (int64_t)g * s_x + (int64_t)b * H * W * C + 4 * c4;
    uint8_t* S = sign + (int64_t)g * s_sign + (int64_t)b * per * c4n + c4;
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    if (stripe < stripes) {
        constexpr int kFly = 8;
        for (int p0 = stripe; p0 < per; p0 += kFly * stripes) {   // kFly positions per thread in flight
            f4 yv[kFly], xv[kFly];
            bool in[kFly];
#pragma unroll
            for (int t = 0; t < kFly; ++t) {
                const int pp = p0 + t * stripes;
                const int yy = (int)fast_div((unsigned)pp, div_wp), xx = pp - yy * Wp;
                in[t] = pp < per && yy >= 1 && yy <= H && xx >= 1 && xx <= W;
                if (in[t]) {
                    yv[t] = __builtin_nontemporal_load((const f4*)(Y + (int64_t)pp * C));
                    xv[t] = __builtin_nontemporal_load((const f4*)(Xs + (int64_t)((yy - 1) * W + (xx - 1)) * C));
                }
            }
#pragma unroll
            for (int t = 0; t < kFly; ++t) {
                const int pp = p0 + t * stripes;
                if (pp >= per) continue;
                unsigned bits = 0;
                if (in[t]) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float a = fmaxf(yv[t][e] + xv[t][e], 0.0f);
                        acc[e] += a;
                        bits |= a > 0.0f ? (1u << e) : 0u;
                    }
                }
                S[(int64_t)pp * c4n] = (uint8_t)bits;
            }
        }
    }
    part[threadIdx.x] = acc;
    __syncthreads();
    if (stripe == 0) {
        for (int s = 1; s < stripes; ++s) acc = acc + part[s * c4n + c4];
        f4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = acc[e] * inv;
        *(f4*)(pooled + (int64_t)g * s_p + (int64_t)b * C + 4 * c4) = o;
    }
}

// dz[g][q][c] = bf16(dpool[g][sample][c] * scale) where the sign bit of (q, c) is set, else 0; dz bf16 padded
constexpr int kPoolBwdFly = 4;   // 16-byte vectors per lane
__global__ __launch_bounds__(kThreads) void pool_bwd_bf16_kernel(const float* __restrict__ dpool, int64_t s_dp,
                                                                 const uint8_t* __restrict__ sign, int64_t s_sign, uint16_t* dz,
                                                                 int64_t s_dz, unsigned vecs, FastDiv div_c8, FastDiv div_pos,
                                                                 int C, float scale) {
    const int g = blockIdx.y;
    const unsigned c8 = (unsigned)C / 8;
    const uint8_t* SG = sign + (int64_t)g * s_sign;
    const float* DP = dpool + (int64_t)g * s_dp;
    u4* DZ = (u4*)(dz + (int64_t)g * s_dz);
    unsigned bits[kPoolBwdFly];
    f4 d0[kPoolBwdFly], d1[kPoolBwdFly];
#pragma unroll
    for (int t = 0; t < kPoolBwdFly; ++t) {   // all the loads of a lane's vectors before the first store
        const unsigned v = (blockIdx.x * kPoolBwdFly + t) * kThreads + threadIdx.x;
        if (v < vecs) {
            const unsigned q = fast_div(v, div_c8);
            const unsigned cv = v - q * c8;
            const unsigned sample = fast_div(q, div_pos);
            bits[t] = *(const uint16_t*)(SG + 2 * (int64_t)v);   // two bytes: channels 8 cv .. 8 cv + 7
            const f4* D = (const f4*)(DP + (int64_t)sample * C) + 2 * cv;
            d0[t] = D[0];
            d1[t] = D[1];
        }
    }
#pragma unroll
    for (int t = 0; t < kPoolBwdFly; ++t) {
        const unsigned v = (blockIdx.x * kPoolBwdFly + t) * kThreads + threadIdx.x;
        if (v >= vecs) continue;
        float o[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o[e] = (bits[t] >> e) & 1u ? d0[t][e] * scale : 0.0f;
            o[4 + e] = (bits[t] >> (8 + e)) & 1u ? d1[t][e] * scale : 0.0f;
        }
        u4 w;   // round to nearest even (v_cvt_pk_bf16_f32)
        w.x = __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{o[0], o[1]}, bf16x2));
        w.y = __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{o[2], o[3]}, bf16x2));
        w.z = __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{o[4], o[5]}, bf16x2));
        w.w = __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{o[6], o[7]}, bf16x2));
        DZ[v] = w;
    }
}

bool aligned16(const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; }

bool shape_ok(const ConvBArgs& a) {
    if (a.groups < 1 || a.groups > 65535 || a.B < 1 || a.H < 1 || a.W < 1 || a.W > kConvBf16MaxWidth || a.C < kCB || a.C % kCB != 0 ||
        a.C > 1024)
        return false;
    const int64_t Pp = (int64_t)a.B * (a.H + 2) * (a.W + 2);
    // 32-bit byte offsets inside one group's bf16 tensor, with room for the rows a tile's strip reaches past either end
    return Pp * a.C < ((int64_t)1 << 31) - (int64_t)1024 * a.C;
}

void fill(ConvBDev* p, const ConvBArgs& a) {
    p->groups = a.groups; p->B = a.B; p->H = a.H; p->W = a.W; p->C = a.C;
    p->Hp = a.H + 2; p->Wp = a.W + 2; p->Pp = a.B * p->Hp * p->Wp; p->halo = p->Wp + 1;
    p->div_per = make_div((unsigned)(p->Hp * p->Wp));
    p->div_wp = make_div((unsigned)p->Wp);
}

// The tile of the forward / delta kernel.  512 pixels x 64 channels where the launch fills the 512 places that two workgroups
// per compute unit make (once, or often enough for the last round not to matter); 256 x 32 where 256 x 64 would leave compute
// units idle; 256 x 64 between them and for strips that do not fit twice (images wider than 49).  us per launch, bf16 output,
// as 512 x 64 / 256 x 64 / 256 x 32:  3 x 20 x 13 x 15 x 128 (30 tiles of 512 pixels) 17.0 / 11.0 / 7.9;  8 x 16 x 24 x 24 x 64 (176)
// 13.1 / 12.3 / 10.8;  4 x 40 x 30 x 30 x 64 (320) 20.9 / 19.1 / 19.8;  8 x 30 x 24 x 32 x 64 (416) 23.8 / 24.6 / 24.9;  12 x 24 x 28 x
// 30 x 64 (540) 31.4 / 29.3 / 32.2;  12 x 60 x 10 x 20 x 128 (744) 55.1 / 58.2 / 63.5;  6 x 64 x 36 x 40 x 64 (1200) 55.1 / 55.3 / 61.1.
struct ConvTile { int tm, tn; };
int strip_pieces(int bm, int W) { return (bm + 2 * (W + 3) + 7) / 8; }
ConvTile conv_tile(int groups, int Pp, int C, int W) {
    const int64_t t512 = (int64_t)groups * ((Pp + 511) / 512) * (C / 64), t256 = (int64_t)groups * ((Pp + 255) / 256) * (C / 64);
    const bool fits = 1024 * strip_pieces(512, W) + (512 + kCB) * 4 <= 80 * 1024;   // two workgroups per compute unit
    if (fits && (t512 >= 680 || (t512 >= 400 && t512 <= 512))) return {4, 2};
    return t256 < 800 ? ConvTile{2, 1} : ConvTile{2, 2};
}

template <int MODE>
hipError_t conv_launch(const ConvBArgs& a, hipStream_t s) {
    const bool tail = MODE == 0 && a.tail;
    if (!shape_ok(a) || !a.in || !a.w || !aligned16(a.in) || !aligned16(a.w)) return hipErrorInvalidValue;
    if (!tail && (!a.out || !aligned16(a.out) || a.s_out % 8)) return hipErrorInvalidValue;
    if (a.s_in % 8 || a.s_w % 8) return hipErrorInvalidValue;
    if (MODE == 1 || (!tail && !a.out_f32)) {   // the sign bytes go with a ReLU's bf16 result and with every delta
        if (!a.gate || !aligned16(a.gate) || a.s_gate % 16 || (MODE == 0 && !a.relu)) return hipErrorInvalidValue;
    }
    if (tail) {   // 16-byte vectors of the shortcut, 32-bit byte offsets in it, at most two samples per 64 padded pixels
        if (a.out_f32 || a.relu || !a.xres || !a.sign || !a.pool_part || !aligned16(a.xres) || !aligned16(a.pool_part) || !aligned16(a.sign) || a.s_x % 4 || a.s_sign % 16 ||
            (a.H + 2) * (a.W + 2) < 64 || (int64_t)a.B * a.H * a.W * a.C >= ((int64_t)1 << 30) - 1024)
            return hipErrorInvalidValue;
    }
    if (MODE == 0 && a.bias && (!aligned16(a.bias) || a.s_bias % 4)) return hipErrorInvalidValue;   // read as 16-byte vectors
    if (MODE == 1 && a.out_f32 && !a.out_unpadded) return hipErrorInvalidValue;   // a padded fp32 delta has no consumer
    if (a.out_unpadded && (!a.out_f32 || tail || (int64_t)a.B * a.H * a.W * a.C >= ((int64_t)1 << 30) - 1024)) return hipErrorInvalidValue;
    if (a.out_f32 && a.relu) return hipErrorInvalidValue;      // the fp32 output is the bare convolution + bias
    ConvBDev p = {};
    fill(&p, a);
    p.in = (const uint16_t*)a.in; p.w = (const uint16_t*)a.w; p.out = a.out;
    p.bias = MODE == 0 ? a.bias : nullptr;
    p.gate = a.gate;
    p.s_in = a.s_in; p.s_w = a.s_w; p.s_out = a.s_out; p.s_bias = a.s_bias; p.s_gate = a.s_gate;
    if (tail) { p.xres = a.xres; p.s_x = a.s_x; p.sign = a.sign; p.s_sign = a.s_sign; p.pool_part = a.pool_part; }
    if (a.stat_part) {
        if (MODE != 0 || !a.out_unpadded || !aligned16(a.stat_part)) return hipErrorInvalidValue;
        p.stat_part = a.stat_part;
    }
    const int out = tail ? kOutTail : a.out_unpadded ? kOutF32U : a.out_f32 ? kOutF32 : kOutBf16;
    if (a.out_f32 && (int64_t)p.Pp * a.C >= ((int64_t)1 << 30)) return hipErrorInvalidValue;   // 32-bit byte offsets in the fp32 output
    if ((int64_t)a.groups * ((p.Pp + 255) / 256) * (a.C / 32) > (1 << 30)) return hipErrorInvalidValue;
    const ConvTile t = conv_tile(a.groups, p.Pp, a.C, a.W);
    const int BM = 128 * t.tm, BN = 32 * t.tn;
    p.tiles_m = (p.Pp + BM - 1) / BM;
    p.tiles_n = a.C / BN;
    p.units = (p.Pp + 255) / 256 * 4;
    p.div_pg = make_div((unsigned)(p.tiles_m * p.tiles_n));
    p.div_tn = make_div((unsigned)p.tiles_n);
    p.total_tiles = a.groups * p.tiles_m * p.tiles_n;
    p.chunk = (p.total_tiles + kXcds - 1) / kXcds;
    p.strip_pieces = strip_pieces(BM, a.W);
    p.strip_bytes = std::max(1024 * p.strip_pieces, stage_bytes(out, BN) + BN * kHalfRows);   // (the gates lie behind the staging)
    const size_t lds = p.strip_bytes + BM * sizeof(int) + BN * sizeof(float);
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    auto pick = [&](auto tm, auto tn) -> void (*)(ConvBDev) {
        constexpr int TM = decltype(tm)::value, TN = decltype(tn)::value;
        if constexpr (MODE == 1) return out == kOutF32U ? conv3x3_bf16_kernel<1, kOutF32U, TM, TN> : conv3x3_bf16_kernel<1, kOutBf16, TM, TN>;
        else return out == kOutTail ? conv3x3_bf16_kernel<0, kOutTail, TM, TN> : out == kOutF32U ? conv3x3_bf16_kernel<0, kOutF32U, TM, TN>
                  : out == kOutF32 ? conv3x3_bf16_kernel<0, kOutF32, TM, TN> : conv3x3_bf16_kernel<0, kOutBf16, TM, TN>;
    };
    typedef std::integral_constant<int, 1> i1;
    typedef std::integral_constant<int, 2> i2;
    typedef std::integral_constant<int, 4> i4;
    void (*kern)(ConvBDev) = t.tm == 4 ? pick(i4(), i2()) : t.tn == 2 ? pick(i2(), i2()) : pick(i2(), i1());
    if (lds > 64 * 1024) {
        hipError_t e = ensure_dynamic_lds((const void*)kern, 160 * 1024);
        if (e != hipSuccess) return e;
    }
    kern<<<(unsigned)(p.chunk * kXcds), kThreads, lds, s>>>(p);
    return hipGetLastError();
}

}  // namespace

#ifdef OLS_CONV_PHASE_PROBE
// dst[3][tiles][8] on the host: the readings of the last launch of each of the three kernels (see conv_phase_probe)
extern "C" __attribute__((visibility("default"))) int ols_debug_conv_phases(unsigned long long* dst, int tiles) {
    if (!dst || tiles < 1 || tiles > kProbeTiles) return -1;
    if (hipDeviceSynchronize() != hipSuccess) return -2;
    for (int k = 0; k < 3; ++k)
        if (hipMemcpyFromSymbol(dst + (size_t)k * tiles * 8, HIP_SYMBOL(conv_phase_probe), (size_t)tiles * 8 * sizeof(unsigned long long),
                                (size_t)k * kProbeTiles * 8 * sizeof(unsigned long long), hipMemcpyDeviceToHost) != hipSuccess)
            return -3;
    return 0;
}
#endif

hipError_t launch_conv3x3_bf16_fwd(const ConvBArgs& a, hipStream_t s) { return conv_launch<0>(a, s); }
hipError_t launch_conv3x3_bf16_dx(const ConvBArgs& a, hipStream_t s) { return conv_launch<1>(a, s); }

namespace {

// One workgroup per compute unit (registers and LDS allow one), so as many ranges as fit one round of the 256 units: one
// more starts a second round for a few workgroups (us per launch, rounded up before: 3 x 64 samples x 36 x 38 x 128, 22 ranges
// 138, 21 83; 9 x 30 x 20 x 20 x 128 72 and 50; 7 x 77 x 2 x 2 x 256 42 and 33).  Past 128 blocks a second round can pay:
// rounds x (slices of a range + what start and end of a workgroup cost, eight slices) + the parts to add up (17 x 14 x 20 x
// 10 x 256, 272 blocks: one range 126, two 115, three 121).
struct DwPlan { int splits; int64_t cost; };
DwPlan dw_plan(int layers, int groups, int B, int H, int W, int C, int64_t most) {   // at most `most` ranges
    const int64_t Pp = (int64_t)B * (H + 2) * (W + 2);
    const int64_t tiles = (int64_t)layers * groups * (C / kCB) * (C / kCB);
    most = std::min(most, (Pp + 511) / 512);                // a range covers at least 512 padded pixels
    int64_t best = 1, best_cost = -1;
    for (int64_t s : {256 / tiles, 512 / tiles, (512 + tiles - 1) / tiles}) {
        if (s > most) s = most;
        if (s < 1) s = 1;
        const int64_t slices = (Pp + s * kDwBK - 1) / (s * kDwBK), rounds = (tiles * s + 255) / 256;
        const int64_t cost = 40 * rounds * (slices + 8) + tiles * s;
        if (best_cost < 0 || cost < best_cost) {
            best = s;
            best_cost = cost;
        }
    }
    return {(int)best, best_cost};
}

bool dw_args_ok(const ConvBArgs& a) {
    return shape_ok(a) && a.in && a.dout && a.partial && a.g && aligned16(a.in) && aligned16(a.dout) && aligned16(a.partial) && a.s_in % 8 == 0 && a.s_dout % 8 == 0;
}

hipError_t dw_launch(const ConvBArgs& a, const ConvBArgs* b, int splits, hipStream_t s) {
    ConvBDev p = {};
    fill(&p, a);
    p.in = (const uint16_t*)a.in; p.dout = (const uint16_t*)a.dout; p.partial = a.partial;
    p.s_in = a.s_in; p.s_dout = a.s_dout;
    if (b) { p.in_b = (const uint16_t*)b->in; p.dout_b = (const uint16_t*)b->dout; p.partial_b = b->partial; }
    p.splits = splits;
    p.k_chunk = (int)(((((int64_t)p.Pp + p.splits - 1) / p.splits) + kDwBK - 1) / kDwBK * kDwBK);
    p.tiles_n = a.C / kCB;
    const int64_t layer = (int64_t)a.groups * p.splits * p.tiles_n * p.tiles_n, total = b ? 2 * layer : layer;
    if (total > (1 << 30)) return hipErrorInvalidValue;
    p.layer_tiles = (int)layer;
    p.total_tiles = (int)total;
    p.chunk = (int)((total + kXcds - 1) / kXcds);
    constexpr size_t lds = kDwFold;
    hipError_t e = ensure_dynamic_lds((const void*)conv3x3_dw_bf16_kernel, lds);
    if (e != hipSuccess) return e;
    conv3x3_dw_bf16_kernel<<<(unsigned)(p.chunk * kXcds), kDwThreads, lds, s>>>(p);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const ConvDwParts parts[2] = {{a.partial, a.g_w_off, a.g_b_off}, b ? ConvDwParts{b->partial, b->g_w_off, b->g_b_off} : ConvDwParts{}};
    return launch_conv_dw_finish(parts, b ? 2 : 1, p.splits, a.groups, a.C, a.g, a.ld, a.guest, s);
}

}  // namespace

int conv3x3_bf16_dw_splits(int groups, int B, int H, int W, int C) { return dw_plan(1, groups, B, H, W, C, INT32_MAX).splits; }

// Two layers in one launch: workgroups start and end once instead of twice, small layers fill compute units that one leaves idle,
// and one finish pass adds up both.  Where the second's sums have no room (many channels on few pixels) two launches stay.  Two
// rounds, us, one state / three in turn: 3 x 20 x 13 x 15 x 128 normalised 670 -> 590 / 485 -> 445 (two launches of 120 workgroups
// took 17.6 each), 9 x 86 x 6 x 13 x 64 plain 501 -> 424 / 407 -> 354, 16 x 128 x 32 x 32 x 64 plain 4503 -> 4430; 24 random
// blocks 1.136 / 1.123 times as fast (1.036 the least).
int conv3x3_bf16_dw_pair_splits(int groups, int B, int H, int W, int C, int64_t scratch_bytes) {
    const int64_t room = scratch_bytes / ((int64_t)groups * (9 * (int64_t)C * C + C) * 4);
    if (room < 1) return 0;
    const DwPlan one = dw_plan(1, groups, B, H, W, C, INT32_MAX), two = dw_plan(2, groups, B, H, W, C, std::min<int64_t>(room, one.splits));
    return two.cost <= 2 * one.cost ? two.splits : 0;
}

hipError_t launch_conv3x3_bf16_dw(const ConvBArgs& a, hipStream_t s) {
    if (!dw_args_ok(a)) return hipErrorInvalidValue;
    return dw_launch(a, nullptr, conv3x3_bf16_dw_splits(a.groups, a.B, a.H, a.W, a.C), s);
}

hipError_t launch_conv3x3_bf16_dw_pair(const ConvBArgs& a, const ConvBArgs& b, int splits, hipStream_t s) {
    if (!dw_args_ok(a) || !dw_args_ok(b) || splits < 1 || a.groups != b.groups || a.B != b.B || a.H != b.H || a.W != b.W || a.C != b.C ||
        a.s_in != b.s_in || a.s_dout != b.s_dout || a.g != b.g || a.ld != b.ld || a.partial == b.partial)
        return hipErrorInvalidValue;
    return dw_launch(a, &b, splits, s);
}

hipError_t launch_pad_cast_bf16(const float* src, int64_t s_src, uint16_t* dst, int64_t s_dst, int groups, int B, int H, int W,
                                int C, const ConvBImages& images, hipStream_t s) {
    if (!src || !dst || groups < 1 || groups > 65535 || B < 1 || H < 1 || W < 1 || C < kCB || C % kCB || !aligned16(src) ||
        !aligned16(dst) || s_src % 4 || s_dst % 8)
        return hipErrorInvalidValue;
    if (images.fwd_a && (!images.wa || !images.wb || !images.fwd_b || !images.dx_b || !aligned16(images.wa) || !aligned16(images.wb) ||
                         !aligned16(images.fwd_a) || !aligned16(images.fwd_b) || !aligned16(images.dx_b) || images.s_w % 8 || images.s_image % 8))
        return hipErrorInvalidValue;
    const int64_t vecs = (int64_t)B * (H + 2) * (W + 2) * (C / 8);
    if (vecs >= ((int64_t)1 << 31) - kPadCastFly * kThreads) return hipErrorInvalidValue;   // the divisions by multiplication take 31-bit dividends
    const int64_t blocks = (vecs + kPadCastFly * kThreads - 1) / (kPadCastFly * kThreads);
    KernelImages im = {{images.wa, images.wb, images.wb}, {images.fwd_a, images.fwd_b, images.dx_b}, images.s_w, images.s_image, C};
    const int64_t image_blocks = images.fwd_a ? 3 * 9 * (int64_t)(C / kCB) * (C / kCB) : 0;
    auto kern = tensors_stream(groups, (int64_t)B * H * W * C) ? pad_cast_bf16_kernel<true> : pad_cast_bf16_kernel<false>;
    kern<<<dim3((unsigned)(blocks + image_blocks), (unsigned)groups), kThreads, 0, s>>>(
        src, s_src, dst, s_dst, (unsigned)vecs, H, W, C, make_div((unsigned)(C / 8)), make_div((unsigned)((H + 2) * (W + 2))),
        make_div((unsigned)(W + 2)), im, (unsigned)image_blocks);
    return hipGetLastError();
}

hipError_t launch_shortcut_relu_pool(const float* y, int64_t s_y, const float* X, int64_t s_x, float* pooled, int64_t s_p,
                                     uint8_t* sign, int64_t s_sign, int groups, int B, int H, int W, int C, hipStream_t s) {
    if (!y || !X || !pooled || !sign || groups < 1 || groups > 65535 || B < 1 || H < 1 || W < 1 || C < 8 || C % 8 || C > 1024 ||
        !aligned16(y) || !aligned16(X) || !aligned16(pooled) || (reinterpret_cast<uintptr_t>(sign) & 1u) || s_y % 4 || s_x % 4 ||
        s_p % 4 || s_sign % 2)
        return hipErrorInvalidValue;
    shortcut_relu_pool_kernel<<<dim3((unsigned)B, (unsigned)groups), kThreads, 0, s>>>(
        y, s_y, X, s_x, pooled, s_p, sign, s_sign, H, W, C, make_div((unsigned)(W + 2)), 1.0f / (float)(H * W));
    return hipGetLastError();
}

int64_t conv3x3_bf16_stat_part_floats(int B, int H, int W, int C) {
    const int64_t Pp = (int64_t)B * (H + 2) * (W + 2);
    return ((Pp + 255) / 256) * 4 * 3 * C;   // per group
}

int64_t conv3x3_bf16_pool_part_floats(int B, int H, int W, int C) {
    const int64_t Pp = (int64_t)B * (H + 2) * (W + 2);
    return ((Pp + 255) / 256) * 4 * 2 * C;   // per group
}

hipError_t launch_pool_bwd_bf16(const float* dpool, int64_t s_dp, const uint8_t* sign, int64_t s_sign, uint16_t* dz, int64_t s_dz,
                                int groups, int B, int positions, int C, float scale, hipStream_t s) {
    if (!dpool || !sign || !dz || groups < 1 || groups > 65535 || B < 1 || positions < 1 || C < 8 || C % 8 || !aligned16(dpool) ||
        (reinterpret_cast<uintptr_t>(sign) & 1u) || !aligned16(dz) || s_dp % 4 || s_sign % 2 || s_dz % 8)
        return hipErrorInvalidValue;
    const int64_t vecs = (int64_t)B * positions * (C / 8);
    if (vecs >= ((int64_t)1 << 31) - kPoolBwdFly * kThreads) return hipErrorInvalidValue;   // the divisions by multiplication take 31-bit dividends
    const int64_t blocks = (vecs + kPoolBwdFly * kThreads - 1) / (kPoolBwdFly * kThreads);
    pool_bwd_bf16_kernel<<<dim3((unsigned)blocks, (unsigned)groups), kThreads, 0, s>>>(
        dpool, s_dp, sign, s_sign, dz, s_dz, (unsigned)vecs, make_div((unsigned)(C / 8)), make_div((unsigned)positions), C, scale);
    return hipGetLastError();
}

}  // namespace ols
