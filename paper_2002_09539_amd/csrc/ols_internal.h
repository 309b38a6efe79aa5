// Internal declarations shared by the translation units of libols (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ols.h"

namespace ols {

// ---------------------------------------------------------------------------------------------
// Launchers.  Each validates its operand shapes on the host and returns a hipError_t; kernels
// themselves live in the matching kernels_*.hip file.  All pointers are device pointers.
// ---------------------------------------------------------------------------------------------

// Whether the kernels that stream over [m][ld] state (local step, with and without the pull-back; step + pull-back + mean;
// stale average) use non-temporal accesses.  Up to 25 million elements, parameters, momenta and gradients are worth leaving in the
// 256 MiB memory-side cache.  Two rounds, non-temporal over plain, by millions of elements (8 workers, momentum 0.9), and the same
// without momentum, where the state is a third smaller and the line could lie higher:
//                          3     9    18    25    30    36    50          3     9    18    25    30    36    50
//   paper     tau 1     1.08  1.06  1.07  1.06  1.03  1.02  0.99       1.03  1.05  1.07  1.06  1.05  1.04  1.01
//             tau 4     1.03  1.09  1.08  1.08  0.98  0.93  0.93       0.99  1.11  1.07  1.07  1.06  1.04  0.98
//   one pass  tau 1     1.03  1.08  1.03  1.07  0.96  0.86  0.87       1.00  1.11  1.11  1.05  1.07  1.06  0.89
//             tau 4     1.13  1.10  1.07  1.08  1.03  0.95  0.92       1.01  1.10  1.09  1.06  1.09  1.08  0.99
//   stale     tau 1     1.00  1.09  1.09  1.00  0.99  0.97  0.96       1.01  1.09  1.12  1.05  1.00  0.98  0.96
//             tau 4     1.06  1.10  1.09  1.06  0.98  0.93  0.93       0.99  1.10  1.09  1.05  1.05  1.02  0.95
//   mixing    tau 1     0.99  1.03  1.08  1.08  1.07  1.02  0.99       0.93  1.00  1.04  1.06  1.06  1.06  1.06
//   (steps)   tau 4     1.09  1.06  1.06  1.08  1.00  0.93  0.93       1.01  1.04  1.05  1.06  1.07  1.07  0.98
// (3 million elements without momentum take 20 to 114 us for all the calls of two rounds: the host's time.)
inline bool state_streams(int64_t m, int64_t ld) { return m * ld > 25000000; }

struct UpdateArgs {
    const float* g;     // [m][ld] gradients
    const float* x_in;  // [m][ld] parameters read
    float* x_out;       // [m][ld] parameters written (may alias x_in)
    float* buf;         // [m][ld] momentum buffers, in place (nullptr iff mu == 0)
    const float* z;     // [ld] anchor, read when pull
    uint16_t* shadow;   // [m][ld] bf16 copy of x_out written in the same pass, or nullptr
    int m;
    int64_t ld;
    float gamma, mu, alpha;
    bool nesterov, pull;
};
hipError_t launch_step(const UpdateArgs& a, hipStream_t s);                      // local step (+ pull-back)
hipError_t launch_pull(float* x, const float* z, uint16_t* shadow, int m, int64_t ld, float alpha,
                       hipStream_t s);                                            // stand-alone pull-back
hipError_t launch_stale_sync(float* x, float* snap, const float* z, uint16_t* shadow, int m, int64_t ld,
                             hipStream_t s);                                      // x <- z + (x - snap); snap <- x
hipError_t launch_init(float* x, float* x_alt, float* buf, float* z, uint16_t* shadow, const float* x0, int m,
                       int64_t d, int64_t ld, hipStream_t s);

struct MeanArgs {
    const float* x;  // [m][ld]
    float* z;        // [ld] anchor (read-modify-write when v != nullptr)
    float* v;        // [ld] anchor momentum buffer or nullptr
    int m;
    int64_t ld;
    float beta_z;
    int split;  // 0 auto, else wavefronts sharing the replica axis (1, 2, 4)
};
hipError_t launch_mean(const MeanArgs& a, hipStream_t s);
int mean_auto_split(int m, int64_t ld);

// step + pull-back + anchor refresh in one pass: one thread owns a column across all replicas
struct StepPullMeanArgs {
    UpdateArgs u;   // u.pull must be true
    float* z_out;   // [ld] new anchor (may alias u.z)
    float* v;       // anchor momentum or nullptr
    float beta_z;
    bool with_step; // false: pull-back + mean only (parameters already stepped)
};
hipError_t launch_step_pull_mean(const StepPullMeanArgs& a, hipStream_t s);
// one wavefront that waits `microseconds` (1 .. 1 000 000) of wall-clock time: emulated communication latency
hipError_t launch_delay(int64_t microseconds, hipStream_t s);

// general mixing X <- X W over the m + 1 rows [x^(1..m), z]
constexpr int kMixMaxWorkers = 128;
struct MixArgs {
    float* x;          // [m][ld] replicas, updated in place
    float* z;          // [ld] anchor (row m of X), updated in place
    uint16_t* shadow;  // [m][ld] bf16 copy of the new replicas, or nullptr
    const float* w;    // [(m + 1)][(m + 1)] row-major on the device
    int m;
    int64_t ld;
};
hipError_t launch_mix(const MixArgs& a, hipStream_t s);

// linear least squares
hipError_t launch_lsq_resid(const float* A, int64_t a_stride, const float* y, int64_t y_stride, const float* x,
                            int64_t ld, float* resid, float* loss_parts, int m, int B, int64_t d, hipStream_t s);
hipError_t launch_lsq_grad(const float* A, int64_t a_stride, const float* resid, float* g, int64_t ld, int m, int B,
                           int64_t d, hipStream_t s);

// Local step (+ pull-back) applied where a gradient element is produced, instead of writing the
// gradient to HBM and streaming it back in a separate pass.  Same fp32 operation sequence as the
// streaming kernels of kernels_update.hip, so both routes give identical bits.
struct FusedUpdate {
    const float* x_in;  // [m][ld] parameters read
    float* x_out;       // [m][ld] parameters written (may alias x_in)
    float* buf;         // [m][ld] momentum buffers (nullptr iff mu == 0)
    const float* z;     // [ld] anchor (pull-back steps)
    uint16_t* shadow;   // [m][ld] bf16 copy of the new parameters, or nullptr
    int64_t ld;
    float gamma, mu, alpha;
    int nesterov, pull;
    int enabled;
    int cached;         // the state is left in the memory-side cache (state_cached)
};
// Whether the arrays that an update reads and writes stay in the 256 MiB memory-side cache until the next one does: both replica
// buffers and `more` bytes per element in 205 MB, which leaves room for the batch and the activations -- or, where rounds of four
// steps or more rewrite one buffer in place most of the time, that buffer and the rest in 185 MB.  (Two arrays in place, alone:
// plain accesses 8.4 - 8.5 TB/s up to 2 x 128 MiB and 5.4 from 2 x 192 MiB on, non-temporal ones 6.1 at every size.)  Two rounds, us,
// non-temporal / plain, batch 64:  9 x (1024-1024-10, bf16), tau 4, 95 MB in place, 551 / 516;  14 x (784-800-400-10), 107 MB, tau 1
// 304 / 283, tau 2 569 / 523, tau 4 1096 / 993;  21 of them, 160 MB, tau 4 1418 / 1363, tau 2 (not taken) 720 / 728;  26 x
// (1024-1024-10), 220 MB (not taken), tau 4 1202 / 1193, 35 of them 1471 / 1514.
inline bool state_cached(int64_t elements, int more, bool in_place) {
    return elements * (8 + more) <= (int64_t)205000000 || (in_place && elements * (4 + more) <= (int64_t)185000000);
}

// Whether a weight gradient with the fused update accesses a layer's state non-temporally (n columns; its weights start w_off
// elements into a replica row).  fp32: only where rows are whole halves of a 128-byte line.  Else two tiles side by side share a
// half, and what the first leaves of it non-temporally does not wait in L2 for the second.  Two rounds, us, three states in turn,
// non-temporal / plain: 30 x (2000-N-10, batch 24) tau 4, N = 1252 3104 / 2765, 1256 2952 / 2745, 1272 2995 / 2775, but 1264 2665 /
// 2750;  40 x (1500-N-10, 48), N = 1036 1382 / 1275, 1032 1330 / 1252, 1048 1340 / 1278, but 1040 1202 / 1251;  29 x (1592-996-14, 32)
// 1108 / 851;  rows that start inside a half: 20 x (1200-648-1024-10, 160) tau 3 2079 / 2003.
// bf16: at any width.  The copy goes out in 2 bytes a weight beside the state's 16, and where the state does not stay in the cache
// plain accesses cost it more than the shared lines: 12 x (3072-N-10, 96) tau 4, N = 656 971 / 1035, 664 1056 / 1064, 648 1058 / 1031;
// 8 x (2048-N-10, 96), N = 2008 686 / 716, 2032 607 / 698;  17 x (944-1264-624-5, 112) 397 / 438;  40 x (3072-216-10, 96) 610 / 649 (with one
// state, which then half fits the cache, N = 648 1218 / 1030 and 43 x (1184-456-13, 96) tau 8 2273 / 1975).
inline bool update_streams(const FusedUpdate& u, int64_t w_off, int n) {
    return !u.cached && (u.shadow || (n % 16 == 0 && w_off % 16 == 0));
}

#if defined(__HIPCC__)
}  // namespace ols
#include "update_rule.h"
namespace ols {
// One element with the anchor value passed in (all operands were fetched ahead of the gradient).
// idx = worker * ld + position inside the replica row.
__device__ __forceinline__ void fused_update_store(const FusedUpdate& u, int64_t idx, float g, float x, float b,
                                                   float z) {
    const bool mom = u.mu != 0.0f;
    const float xn = local_step_elem(g, x, b, z, u.gamma, u.mu, u.alpha, mom, u.nesterov != 0, u.pull != 0);
    if (mom) u.buf[idx] = b;
    u.x_out[idx] = xn;
    if (u.shadow) u.shadow[idx] = (uint16_t)bf16_bits_rne(xn);
}
// The same with the anchor read here (col = position inside the replica row).
__device__ __forceinline__ void fused_update_apply(const FusedUpdate& u, int64_t idx, int64_t col, float g, float x,
                                                   float b) {
    fused_update_store(u, idx, g, x, b, u.pull ? u.z[col] : 0.0f);
}
#endif

// least squares, small problems: residual, loss, gradient and the local step of one or several steps in one launch, with
// the pull-back (u.pull) and the anchor average (with_mean) behind the last of them
bool lsq_step_fits(int B, int64_t d);
// whether the next `steps` steps are faster in one launch (which averages the replicas as well) than in one each
bool lsq_round_pays(int B, int64_t d, int64_t steps, bool with_mean);
bool lsq_round_with_mean(int m, int64_t d, int64_t ld);   // whether with_mean takes m replicas of d parameters, ld apart
struct LsqRoundArgs {
    const float* A;          // batch 0 of worker 0: [nb][B][d] per worker
    const float* y;
    int64_t a_stride, y_stride;   // elements between workers
    int nb, first_batch, steps;   // step t reads batch (first_batch + t) mod nb
    float* loss_parts;
    int m, B;
    int64_t d;
    int with_mean, mean_split;
    unsigned long long* flags;    // [m], any contents (with_mean)
    float* z;                     // (with_mean)
};
hipError_t launch_lsq_round(const LsqRoundArgs& a, const FusedUpdate& u, hipStream_t s);

struct HeadArgs;

// grouped GEMMs over the m workers (group strides in elements)
struct GemmArgs {
    const void* a;      // operand A, group stride sa
    const void* b;      // operand B, group stride sb
    void* c;            // output, group stride sc
    void* a_rounded;    // bf16 fwd of a small launch (gemm_small_bf16_fits), optional: a is fp32, and its bf16 values, which the
                        // product takes, go here as well ([M][K] per group)
    const float* bias;  // fwd: [N] per group, stride sbias
    const void* mask;   // dA: activations whose sign gates the output, same shape as c, stride smask
    float* colsum;      // dw: optional [N] per group, receives the column sums of B (the bias gradient)
    float* partial;     // fp32 fwd with splits > 1: scratch of splits * groups * M * N floats
    int k_chunk;        // split forward with splits > 1: contraction indices of a range, a multiple of 32 (0: an even share)
    int strip_order;    // split forward: add up the products as the column strips do (MlpStripNext)
    int splits;         // fp32 fwd: number of K ranges contracted by separate workgroups (<= 1: none)
    int force_general;  // use the bounds-checked kernel even where the full-tile kernel applies
    const HeadArgs* guest;  // dw: the output layer's weight / bias gradients (launch_head_bwd's work) are computed by
                            // extra workgroups at the front of this launch; nullptr: none
    FusedUpdate upd;    // dw: when enabled, c is NOT written; the update of W (c's position in the replica row is
    int64_t upd_w_off;  //     upd_w_off) and of the bias (upd_b_off, from the column sums) is applied instead
    int64_t upd_b_off;
    int64_t sa, sb, sc, sbias, smask, scolsum;
    int groups;
    int M, N, K;        // output M x N, contraction length K
    int lda, ldb, ldc;  // leading dimensions (elements) of the operands as stored
};
// fp32 MFMA.  fwd: C[M][N] = relu(A[M][K] W[K][N] + bias);  dw: C[M][N] = A[K][M]^T B[K][N];
// da: C[M][N] = (A[M][K] B[N][K]^T) * (mask > 0)
hipError_t launch_gemm_f32_fwd(const GemmArgs& g, hipStream_t s, int variant);
hipError_t launch_gemm_f32_dw(const GemmArgs& g, hipStream_t s, int variant);
hipError_t launch_gemm_f32_da(const GemmArgs& g, hipStream_t s, int variant);
hipError_t launch_splitk_finish(const float* partial, int splits, const GemmArgs& g, hipStream_t s);
// forward and delta of small launches (kernels_gemm_small.hip; gemm_f32_plan.h: whether an fp32 shape takes them)
hipError_t launch_gemm_small_fwd(const GemmArgs& g, hipStream_t s);
hipError_t launch_gemm_small_da(const GemmArgs& g, hipStream_t s);
bool gemm_small_bf16_fits(const GemmArgs& g, bool fwd);
hipError_t launch_gemm_small_bf16_fwd(const GemmArgs& g, hipStream_t s);
hipError_t launch_gemm_small_bf16_da(const GemmArgs& g, hipStream_t s);
// forward on the bf16 matrix cores with every operand split exactly into three bf16 terms (fp32 accuracy)
hipError_t launch_gemm_split_fwd(const GemmArgs& g, hipStream_t s);
// Weight gradient of an fp32 MLP's first hidden layer by column strips (kernels_mlp_strip.hip); with the fused update it can form
// the next step's forward product as well.  Whether a shape takes it, and over how many ranges of the weights' rows: mlp_strip_plan.h.
struct MlpStripNext {
    const float* x;       // the next step's batch, strides as GemmArgs::a
    float* out;           // relu(x W + bias) with the updated parameters, [B][N] per worker
    float* partial;       // ranges > 1: ranges * groups * B * N floats
    const float* bias;    // where the update leaves the bias, upd.ld between workers
    int ranges;
};
hipError_t launch_mlp_strip(const GemmArgs& g, const MlpStripNext* next, hipStream_t s);
// The weight gradients of n layers with the fused update, whose deltas are all there: up to kDwMostLayers in a launch, the bits of
// one launch each.  Only the first may have a guest.
constexpr int kDwMostLayers = 4;
hipError_t launch_gemm_f32_dw_layers(const GemmArgs* g, int n, hipStream_t s);
hipError_t launch_gemm_bf16_dw_layers(const GemmArgs* g, int n, hipStream_t s);
// bf16 operands, fp32 accumulate.  fwd: A[M][K], W[K][N];  dw: A[K][M], B[K][N] (K = batch);  da: A[M][K], W[N][K]
hipError_t launch_gemm_bf16_fwd(const GemmArgs& g, hipStream_t s);
hipError_t launch_gemm_bf16_dw(const GemmArgs& g, hipStream_t s, int variant);
hipError_t launch_gemm_bf16_da(const GemmArgs& g, hipStream_t s);
hipError_t launch_cast_bf16(const float* src, int64_t src_stride, uint16_t* dst, int groups, int rows, int cols,
                            hipStream_t s);

// output layer (N = classes <= 32) on plain vector ALUs
// Partial sums of a fused tail per 64 consecutive pixels, [group][w][2][SUMS][C] (slot 0: the sample of pixel 64 w, slot 1: the
// next one), with `per` (>= 64) pixels per sample; launch_head_fwd adds them up into its h first.
struct PoolParts {
    const float* part;    // nullptr: h is there
    int64_t s_part;       // floats between groups
    float* more;          // SUMS = 3: the sums after the first, [group][2][sample][C]; nullptr: SUMS = 1
    int per;
    float inv;            // h = inv * the first sum
};
struct HeadArgs {
    PoolParts pool;       // launch_head_fwd, fp32 h
    const void* h;        // [m][B][H] last hidden activations (fp32, or bf16 when h_bf16)
    int64_t h_stride;     // elements between workers in h
    bool h_bf16;
    const float* x;       // [m][ld] parameters; W_L at w_off, b_L at b_off within a row
    float* g;             // [m][ld] gradients, same offsets
    int64_t ld, w_off, b_off;
    const int32_t* labels;
    int64_t label_stride;
    float* dlogits;       // [m][B][C]
    float* loss_parts;    // [m][B] per-sample losses
    void* dz;             // [m][B][H] delta for the last hidden layer (fp32 or bf16), masked by h > 0
    int m, B, H, C;
    FusedUpdate upd;      // when enabled the output layer's parameters are updated instead of writing g
};
hipError_t launch_head_fwd(const HeadArgs& a, hipStream_t s);
hipError_t launch_head_bwd(const HeadArgs& a, hipStream_t s);
// Whether the block's streaming kernels read activation tensors of groups x elements floats non-temporally: above 48 MB each.
// Two rounds, non-temporal over plain, bf16 normalised blocks by MB per tensor: 8: 1.05, 14: 1.06, 16: 1.06, 29: 1.06, 35: 1.05, 42:
// 1.01, 57: 0.99, 76: 1.01, 120: 1.00.
inline bool tensors_stream(int64_t groups, int64_t elements) { return groups * elements * 4 > 48000000; }

// 3 x 3 convolutions (stride 1, zero padding 1) grouped over the workers; activations [group][B H W][C] (channel
// contiguous), kernels [group][9][C][C] as (tap, input channel, output channel).  C a multiple of 16.
struct ConvArgs {
    const float* in;        // fwd: layer input; dx: delta of the layer output; dw: layer input
    const float* w;         // fwd, dx: kernels
    const float* dout;      // dw: delta of the layer output
    float* out;             // fwd: layer output; dx: delta of the layer input
    const float* bias;      // fwd: [C] per group, or nullptr for a convolution without bias
    const float* residual;  // fwd: added before the activation (same shape as out), or nullptr
    const float* mask;      // dx: activations whose sign gates the result (same shape as out), or nullptr
    float* partial;         // dw: scratch of dw_splits * groups * (9 C C + C) floats
    int dw_splits;          // dw: pixel ranges the contraction is split into
    float* g;               // dw: gradients [groups][ld]; kernel gradient at g_w_off, bias gradient at g_b_off of a row
                            // (g_b_off < 0: no bias, nothing written for it)
    int64_t ld, g_w_off, g_b_off;
    const HeadArgs* guest;  // dw, optional: the classifier's gradients (launch_head_bwd's work), in the finish pass's launch
    int64_t s_in, s_w, s_dout, s_out, s_bias, s_res, s_mask;   // group strides (elements)
    int groups, B, H, W, C;
    int relu;               // fwd: apply max(., 0)
    // split kernels (launch_conv3x3_split_weights), set where conv3x3_split_fits: fwd resp. dx reads these in place of w
    const uint8_t* w_split;
    const uint8_t* w_split_dx;
    // split fwd, optional, C a multiple of 64: [group][conv3x3_split_stat_parts(...)][3][C] statistics of the output per
    // tile of pixels (count, mean, sum of squared deviations) for BnArgs::wave_part
    float* stat_part;
};
hipError_t launch_conv3x3_fwd(const ConvArgs& a, hipStream_t s);
hipError_t launch_conv3x3_dx(const ConvArgs& a, hipStream_t s);
hipError_t launch_conv3x3_dw(const ConvArgs& a, hipStream_t s);   // weight + bias gradient (two launches)
int conv3x3_dw_splits(int groups, int B, int H, int W, int C, int least = 256);   // pixel ranges (of `least` at least) the weight-gradient contraction is split into
// The same products on the bf16 matrix cores with every fp32 operand split exactly into three bf16 terms (fp32 accuracy);
// the kernels are split once per step: forward images of both, delta image of the second (dst: weight_bytes(groups) each).
bool conv3x3_split_fits(int B, int H, int W, int C);
int64_t conv3x3_split_weight_bytes(int groups, int C);
int64_t conv3x3_split_stat_parts(int B, int H, int W);
hipError_t launch_conv3x3_split_weights(const float* wa, const float* wb, uint8_t* fwd_a, uint8_t* fwd_b, uint8_t* dx_b,
                                        int64_t s_w, int groups, int C, hipStream_t s);
hipError_t launch_conv3x3_split_fwd(const ConvArgs& a, hipStream_t s);
hipError_t launch_conv3x3_split_dx(const ConvArgs& a, hipStream_t s);
hipError_t launch_conv3x3_split_dw(const ConvArgs& a, hipStream_t s);   // (two launches)
int conv3x3_split_dw_splits(int groups, int B, int H, int W, int C);
// second pass of the kernel gradients of one or two layers: sums the pixel ranges' parts [splits][groups][9 C C + C] in range
// order into g
struct ConvDwParts {
    const float* partial;
    int64_t w_off, b_off;   // b_off < 0: no bias
};
hipError_t launch_conv_dw_finish(const ConvDwParts* layers, int n, int splits, int groups, int C, float* g, int64_t ld,
                                 const HeadArgs* guest, hipStream_t s);
// pooled = scale * sum over the HW positions of every sample (scale = 1 / HW: global average pooling), and the backward
// of the average through the ReLU in front of it
hipError_t launch_pool_mean(const float* a, int64_t s_a, float* pooled, int64_t s_p, int groups, int B, int HW, int C,
                            float scale, hipStream_t s);
hipError_t launch_pool_bwd(const float* dpool, int64_t s_dp, const float* a, int64_t s_a, float* dz, int64_t s_dz,
                           int groups, int B, int HW, int C, hipStream_t s);

// The same convolutions with bf16 operands.  Operand tensors carry their zero border: [group][B (H+2) (W+2)][C] bf16,
// channel contiguous.  C a multiple of 64, W at most kConvBf16MaxWidth.
constexpr int kConvBf16MaxWidth = 128;
struct ConvBArgs {
    const void* in;         // fwd: layer input; dx: delta of the layer output; dw: layer input (bf16, padded)
    const void* w;          // fwd, dx: bf16 kernels, an image of launch_pad_cast_bf16
    const void* dout;       // dw: delta of the layer output (bf16, padded)
    void* out;              // fwd: layer output; dx: delta of the layer input; padded, bf16 -- or, fwd with out_f32, the
                            // bare convolution + bias in fp32 with border rows as computed (their consumer skips them)
    int out_f32;
    int out_unpadded;       // with out_f32 (fwd and dx): fp32 [B H W][C], image pixels only -- what a batch normalisation reads
    float* stat_part;       // fwd with out_unpadded, optional: conv3x3_bf16_stat_part_floats(...) floats per group; per 64
                            // padded pixels (count, mean, sum of squared deviations) [3][C] of the output's image pixels,
                            // which launch_bn_forward takes instead of reading the output for its statistics
    const float* bias;      // fwd: [C] per group, or nullptr
    uint8_t* gate;          // dx: [row of the output][C / 4] sign bytes (bit e set: channel 4 c + e stays, else 0); fwd with
                            // bf16 output: where the output leaves its own (bit e set iff it is positive)
    const void* mask;       // launch_conv3x3_bf16_slices_dx: the padded bf16 activations whose sign gates the result
    float* partial;         // dw: scratch of conv3x3_bf16_dw_splits(...) * groups * (9 C C + C) floats
    float* g;               // dw: gradients [groups][ld]
    int64_t ld, g_w_off, g_b_off;   // g_b_off < 0: no bias
    const HeadArgs* guest;  // dw, optional: the classifier's gradients (launch_head_bwd's work), in the finish pass's launch
    int64_t s_in, s_w, s_dout, s_out, s_bias, s_gate, s_mask;   // group strides (elements of the tensor's own type)
    int groups, B, H, W, C;
    int relu;               // fwd with bf16 output: max(., 0) is applied, and has to be asked for
    // fwd with the residual block's tail fused in (tail != 0; out unused, no relu, padded images of at least 64 pixels):
    // a2 = relu(convolution + bias + xres) is never stored -- sign[padded pixel][C / 4] gets one byte per four channels
    // with bit e set iff a2 > 0 (border: 0), and pool_part (conv3x3_bf16_pool_part_floats(...) floats per group) the
    // partial sums that launch_head_fwd turns into the mean over the positions (PoolParts).
    int tail;
    const float* xres;      // fp32 [B H W][C], not padded
    uint8_t* sign;
    float* pool_part;
    int64_t s_x, s_sign;    // group strides
};
hipError_t launch_conv3x3_bf16_fwd(const ConvBArgs& a, hipStream_t s);
hipError_t launch_conv3x3_bf16_dx(const ConvBArgs& a, hipStream_t s);
hipError_t launch_conv3x3_bf16_dw(const ConvBArgs& a, hipStream_t s);
// the plain block's forward (bf16 output or fused tail) and delta in launches of middling size, and whether a shape takes them:
// w is the bf16 kernels themselves, there are no sign bytes of the output, and the delta is gated by `mask`
bool conv3x3_bf16_slices_fits(int groups, int B, int H, int W, int C);
hipError_t launch_conv3x3_bf16_slices_fwd(const ConvBArgs& a, hipStream_t s);
hipError_t launch_conv3x3_bf16_slices_dx(const ConvBArgs& a, hipStream_t s);
int conv3x3_bf16_dw_splits(int groups, int B, int H, int W, int C);
// the kernel gradients of two layers of one shape in one launch: its pixel ranges, each layer's `partial` as large as they make
// it (the second layer's in scratch_bytes, the first's never larger than for conv3x3_bf16_dw_splits), or 0: two launches instead
int conv3x3_bf16_dw_pair_splits(int groups, int B, int H, int W, int C, int64_t scratch_bytes);
hipError_t launch_conv3x3_bf16_dw_pair(const ConvBArgs& a, const ConvBArgs& b, int splits, hipStream_t s);
int64_t conv3x3_bf16_pool_part_floats(int B, int H, int W, int C);   // per group
int64_t conv3x3_bf16_stat_part_floats(int B, int H, int W, int C);   // per group
// The step's kernels in fragment order, which launch_conv3x3_bf16_fwd / _dx take as ConvBArgs::w: 9 C C values per group for the
// first convolution, the second, and the second's delta.  All nullptr: none are made.
struct ConvBImages {
    const uint16_t *wa, *wb;             // bf16 kernels [9][C][C] per group
    uint16_t *fwd_a, *fwd_b, *dx_b;
    int64_t s_w, s_image;                // group strides
};
// fp32 [groups][B H W][C] -> bf16 [groups][B (H+2) (W+2)][C] with a zero border; and the images of the step's kernels
hipError_t launch_pad_cast_bf16(const float* src, int64_t s_src, uint16_t* dst, int64_t s_dst, int groups, int B, int H, int W,
                                int C, const ConvBImages& images, hipStream_t s);
// The block's tail: a2 = relu(y + X) on the image pixels (y fp32 padded, X fp32 not padded), pooled = its mean over the
// positions, sign[padded pixel][C / 4] = one byte per four channels with bit e set iff a2 > 0 (border: 0).  a2 is not stored.
hipError_t launch_shortcut_relu_pool(const float* y, int64_t s_y, const float* X, int64_t s_x, float* pooled, int64_t s_p,
                                     uint8_t* sign, int64_t s_sign, int groups, int B, int H, int W, int C, hipStream_t s);
// dz = bf16(dpool * scale) where the sign bit is set, else 0; dz bf16 over `positions` (padded) positions per sample
hipError_t launch_pool_bwd_bf16(const float* dpool, int64_t s_dp, const uint8_t* sign, int64_t s_sign, uint16_t* dz, int64_t s_dz,
                                int groups, int B, int positions, int C, float scale, hipStream_t s);

// Batch normalisation in training mode over [group][P][C] tensors (statistics per group and channel over the P pixels).
struct BnArgs {
    const float* z;         // convolution output
    float* out;             // fwd: act(gamma xhat + beta (+ shortcut))
    const float* shortcut;  // fwd: added before the activation, or nullptr
    float* dy;              // bwd: gradient at the normalised output on entry, gradient at z on return (in place)
    float* stats;           // [group][2][C]: mean, 1 / sqrt(var + eps); written by fwd, read by bwd
    float* sums;            // bwd: [group][2][C] scratch (sum dy, sum dy xhat)
    float* part;            // scratch of bn_partial_floats(...) floats
    const float* gamma;     // scale, [C] per group
    const float* beta;      // shift (fwd)
    float* g;               // bwd: gradients [groups][ld]; d gamma at g_gamma_off, d beta at g_beta_off of a row
    int64_t ld, g_gamma_off, g_beta_off;
    int64_t s_z, s_out, s_sc, s_dy, s_par;   // group strides (elements); s_par for gamma and beta
    int groups, P, C;
    int relu;
    float eps;
    // Optional: the result (fwd: the activation; bwd: the gradient at z) goes out as bf16, to nearest even, in the padded
    // operand layout of the bf16 convolutions, [B (H + 2) (W + 2)][C] per group with P = B H W -- only the image pixels
    // are written (the border is zero from the start and stays so); `out` / the in-place update of dy are then skipped.
    // (fwd) `gate_out`, with out_bf16: [P][C / 4] sign bytes of the bf16 result (bit e set iff channel 4 c + e is positive).
    uint16_t* out_bf16;
    int64_t s_outb;
    int H, W;
    uint8_t* gate_out;
    int64_t s_gate_out;
    // Optional (bwd): the normalised output sits under a ReLU and global average pooling, so the gradient on entry is
    // dpool[group][sample][c] / positions where gate (the activation, [group][P][C]) is positive and 0 elsewhere; it is
    // formed on the fly and dy is only written (the gradient at z), or not touched at all with out_bf16.
    const float* gate;
    const float* dpool;
    int64_t s_gate, s_dp;
    int positions;
    // Optional (fwd): partial statistics that the producer of z left (ConvBArgs / ConvArgs::stat_part), [group][waves][3][C]:
    // the statistics are merged from them and z is read only once, by the normalisation itself.
    const float* wave_part;
    int waves;
    // Optional (fwd, with shortcut / relu as given; H * W >= 64): the block's tail.  The activation is not stored: `sign`
    // gets one byte per pixel and four channels ([group][P][C / 4], bit e set iff the activation is positive) and
    // `pool_part` ([group][ceil(P / 64)][2][3][C] floats) per 64 pixels the activation's sums, the number of positive
    // activations and their sums of xhat, for PoolParts (with `more`).
    // (bwd) `sign` in place of `gate`: the same bytes say where the activation was positive; `sample_sums`
    // ([group][2][sample][C]: numbers and sums of xhat, PoolParts' `more`) then has to be given.
    uint8_t* sign;
    float* pool_part;
    const float* sample_sums;
    int64_t s_sign;
};
hipError_t launch_bn_forward(const BnArgs& a, hipStream_t s);    // statistics (one or two launches) + normalise
hipError_t launch_bn_backward(const BnArgs& a, hipStream_t s);   // sums (two launches) + gradient at z
int64_t bn_partial_floats(int groups, int P, int C);

// raises a kernel's dynamic-LDS limit once per (device, kernel)
hipError_t ensure_dynamic_lds(const void* kernel, size_t bytes);
inline int64_t round_up(int64_t v, int64_t q) { return (v + q - 1) / q * q; }

}  // namespace ols
