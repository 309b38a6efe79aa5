// Output layer of the per-worker MLP (class count C <= 32) with softmax cross-entropy, the delta it
// sends back to the last hidden layer, and its own gradients.  They are a few MFLOP per worker: what they cost is
// (a) the chain of dependent memory round trips and (b) instruction fetch -- a launch this small runs
// every instruction a handful of times, so long unrolled code is paid for line by line from a cold
// instruction cache.
//
//   head_fwd_kernel   logits, loss, dlogits AND the hidden delta dz in one launch.  Both products run on the fp32 matrix
//                     cores (v_mfma_f32_16x16x4_f32) on fragments loaded straight into registers: a workgroup owns 16
//                     samples, its wavefronts share the hidden units out, and everything the launch reads -- activations,
//                     weights in both fragment orders, labels -- is requested in one round trip; the activations stay in
//                     registers as the ReLU mask of dz.
//   head_dw_kernel    dW = h^T dlogits, db = colsum(dlogits), consumed by the fused update or stored (body in
//                     head_dw_body.h; by default it runs as guest workgroups of a weight-gradient GEMM instead).
//
// Per worker i with last hidden activations h [B][H], weights W [H][C], bias b [C], labels y [B]
// (the mini-batch loss whose gradient is the g_i of Section 2, arXiv 2002.09539):
//   logits = h W + b;  loss_s = logsumexp(logits_s) - logits_s[y_s];  dlogits = (softmax - onehot) / B
//   dW = h^T dlogits;  db = colsum(dlogits);  dz = (dlogits W^T) * [h > 0]
// The class dimension is padded to CMAX (16 or 32) with zeros so that no inner loop branches on C.
#include "gemm_bf16_tile.h"
#include "head_dw_body.h"
#include "ols_internal.h"

namespace ols {

constexpr int kRow = 16;     // lanes of one DPP row
constexpr int kMaxC = 32;

__device__ __forceinline__ unsigned int f32_to_bf16(float f) { return bf16_bits_rne(f); }
// Sum over the 16 lanes of a DPP row, the same bits in every lane of the row (each step adds a lane's
// value to that of its partner 8, 4, 2, 1 lanes away, which is symmetric).
__device__ __forceinline__ float row_sum(float v) {
#define OLS_ROW_ROR_ADD(n)                                                                                  \
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + (n), 0xF, 0xF, false))
    OLS_ROW_ROR_ADD(8);
    OLS_ROW_ROR_ADD(4);
    OLS_ROW_ROR_ADD(2);
    OLS_ROW_ROR_ADD(1);
#undef OLS_ROW_ROR_ADD
    return v;
}

__device__ __forceinline__ float row_max(float v) {
#define OLS_ROW_ROR_MAX(n)                                                                                  \
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + (n), 0xF, 0xF, false)))
    OLS_ROW_ROR_MAX(8);
    OLS_ROW_ROR_MAX(4);
    OLS_ROW_ROR_MAX(2);
    OLS_ROW_ROR_MAX(1);
#undef OLS_ROW_ROR_MAX
    return v;
}

struct HeadDev {
    const void* h;
    const float* x;
    const int32_t* labels;
    float* dlogits;
    float* loss_parts;
    void* dz;
    int64_t h_stride, ld, w_off, b_off, label_stride;
    int B, H, C;
    PoolParts pool;
};

// A block's pooled features from the partial sums that its fused tail left: pooled[n][c] = inv * the sum for sample n.  Part w
// covers the pixels 64 w .. 64 w + 63 (padded pixels for the convolution's tail, image pixels for the normalisation's), its first
// sample is floor(64 w / per) with per pixels per sample, and its two slots are that sample and the next.  A slot holds SUMS sums of
// C channels; those after the first go to more[SUMS - 1][n][c] as they are.  Added in order of w; one lane per (sample, channel quad).
// The workgroup that classifies a sample adds up its parts; as a launch of its own that took 4 to 9 us.  Two rounds, us: plain
// 4 x 17 x 13 x 13 x 64 295 -> 284, 12 x 8 x 9 x 14 x 64 tau 3 441 -> 427, normalised 3 x 12 x 35 x 36 x 64 589 -> 581; 16 random bf16 blocks
// 1.014 times as fast (0.995 the least).
template <int SUMS>
__device__ __forceinline__ void pool_finish(const HeadDev& p, int i, int n, int c4) {
    const int C = p.H, c4n = C / 4, per = p.pool.per;
    const f4* P = (const f4*)(p.pool.part + (int64_t)i * p.pool.s_part) + c4;
    const int w_lo = (n * per) / 64, w_hi = ((n + 1) * per - 1) / 64;
    f4 acc[SUMS];
#pragma unroll
    for (int k = 0; k < SUMS; ++k) acc[k] = f4{0.f, 0.f, 0.f, 0.f};
    constexpr int kFly = 8;   // the loads of eight parts ahead of their additions
    for (int w0 = w_lo; w0 <= w_hi; w0 += kFly) {
        f4 v[kFly][SUMS];
#pragma unroll
        for (int t = 0; t < kFly; ++t) {
            const int w = w0 + t <= w_hi ? w0 + t : w_hi;
            const int slot = n - (64 * w) / per;   // 0 or 1
#pragma unroll
            for (int k = 0; k < SUMS; ++k) v[t][k] = P[((int64_t)(2 * w + slot) * SUMS + k) * c4n];
        }
#pragma unroll
        for (int t = 0; t < kFly; ++t)
            if (w0 + t <= w_hi) {
#pragma unroll
                for (int k = 0; k < SUMS; ++k) acc[k] = acc[k] + v[t][k];
            }
    }
    f4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = acc[0][e] * p.pool.inv;
    *(f4*)((float*)p.h + (int64_t)i * p.h_stride + (int64_t)n * C + 4 * c4) = o;
#pragma unroll
    for (int k = 1; k < SUMS; ++k) *(f4*)(p.pool.more + (((int64_t)i * (SUMS - 1) + k - 1) * p.B + n) * C + 4 * c4) = acc[k];
}

// Measured against a kernel that staged weights and activations in LDS and formed both products on the vector ALUs, us per
// launch: 14.9 -> 12.0 (16 workers x 128 samples x 512 units), 27.9 -> 18.0 (64 x 64 x 1024), 52.7 -> 24.1 (16 x 256 x 2048, bf16),
// 12.1 -> 8.5 (5 x 36 x 124).
// A wavefront takes T tiles of 16 hidden units per pass; layers wider than WAVES T 16 units take several passes and read
// activations and weights again for dz.
// Fragment layout of the 16x16x4 product: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]; register r of the result is
// [4 (l / 16) + r][l % 16].  Logits: A = h (rows samples), B = W; product e of a tile contracts the units 4 (l / 16) + e, so
// a lane's four products take one 4-wide vector of its sample.  dz: A = W (rows units), B = dlogits^T, so a lane's result is
// four consecutive units of sample l % 16 -- the units whose activations it holds.
constexpr unsigned kHeadNowhere = 0x80000000u;   // beyond every range, also with a tile's offset added

// grid (ceil(B / 16), m)
template <bool BF, int CMAX, int T, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void head_fwd_kernel(HeadDev p) {
    constexpr int S = 16, CT = CMAX / 16, CS = CMAX / 4, kChunk = WAVES * T * 16;
    __shared__ float s_part[WAVES][S * CMAX];   // the wavefronts' shares of the logits
    __shared__ float s_d[S][CMAX + 1];
    const int C = p.C, H = p.H, B = p.B;
    const int i = blockIdx.y, s0 = blockIdx.x * S;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, l16 = lane % 16, q = lane / 16;
    const int rows = min(S, B - s0);
    const unsigned es = BF ? 2u : 4u;
    const rsrc_t h_rs = make_rsrc((const char*)p.h + ((int64_t)i * p.h_stride + (int64_t)s0 * H) * es, (unsigned)rows * (unsigned)H * es);
    const rsrc_t w_rs = make_rsrc(p.x + (int64_t)i * p.ld + p.w_off, 4u * (unsigned)H * (unsigned)C);
    auto w_at = [&](unsigned off) { return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(w_rs, (int)off, 0, 0)); };

    // the softmax's operands: lane (sample threadIdx / 16, class threadIdx % 16) of the first four wavefronts
    const int row = threadIdx.x / kRow, sub = threadIdx.x % kRow, s = s0 + row;
    const bool soft = threadIdx.x < S * kRow, live = soft && s < B;
    float bias[CT];
#pragma unroll
    for (int c0 = 0; c0 < CT; ++c0) bias[c0] = soft && kRow * c0 + sub < C ? p.x[(int64_t)i * p.ld + p.b_off + kRow * c0 + sub] : 0.0f;
    const int label = live ? p.labels[(int64_t)i * p.label_stride + s] : 0;

    if constexpr (!BF) {
        if (p.pool.part) {   // the workgroup's own samples; its loads of them below come behind the barrier
            for (int v = threadIdx.x; v < rows * (H / 4); v += 64 * WAVES) {
                const int n = v / (H / 4), c4 = v - n * (H / 4);
                if (p.pool.more) pool_finish<3>(p, i, s0 + n, c4);
                else pool_finish<1>(p, i, s0 + n, c4);
            }
            __syncthreads();
        }
    }

    f4 hv[BF ? 1 : T];
    u2 hb[BF ? T : 1];
    float w1[T][4][CT], w2[T][CS];
    auto load_h = [&](int k0) {   // units k0 + 16 t + 4 q .. + 3 of sample l16 (zeros past the layer and past the batch)
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int k = k0 + 16 * t + 4 * q;
            const unsigned off = k < H ? ((unsigned)l16 * (unsigned)H + (unsigned)k) * es : kHeadNowhere;
            if constexpr (BF) hb[t] = __builtin_bit_cast(u2, __builtin_amdgcn_raw_buffer_load_b64(h_rs, (int)off, 0, 0));
            else hv[t] = __builtin_bit_cast(f4, buf_load(h_rs, off, 0u));
        }
    };
    auto h_elem = [&](int t, int e) {
        if constexpr (BF) return head_bf16_elem(e < 2 ? hb[t].x : hb[t].y, e);
        else return hv[t][e];
    };
    auto load_w1 = [&](int k0) {   // W[k0 + 16 t + 4 q + e][16 j + l16]
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const unsigned first = 16 * j + l16 < C ? 4u * ((unsigned)(k0 + 4 * q) * (unsigned)C + 16u * j + l16) : kHeadNowhere;
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) w1[t][e][j] = w_at(first + 4u * (unsigned)((16 * t + e) * C));
        }
    };
    auto load_w2 = [&](int k0) {   // W[k0 + 16 t + l16][4 c + q]
#pragma unroll
        for (int c = 0; c < CS; ++c) {
            const unsigned first = 4 * c + q < C ? 4u * ((unsigned)(k0 + l16) * (unsigned)C + 4u * c + q) : kHeadNowhere;
#pragma unroll
            for (int t = 0; t < T; ++t) w2[t][c] = w_at(first + 64u * (unsigned)(t * C));
        }
    };

    const bool one_pass = H <= kChunk;
    f4 acc[CT];
#pragma unroll
    for (int j = 0; j < CT; ++j) acc[j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int c0 = 0; c0 < H; c0 += kChunk) {
        const int k0 = c0 + wave * T * 16;
        load_h(k0);
        load_w1(k0);
        if (one_pass && p.dz) load_w2(k0);
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < CT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(h_elem(t, e), w1[t][e][j], acc[j], 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < CT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) s_part[wave][(4 * q + r) * CMAX + 16 * j + l16] = acc[j][r];
    __syncthreads();
    if (soft) {
        // Softmax with the classes spread over the 16 lanes of the row: lane sub owns class sub (and sub + 16 when CMAX =
        // 32), so each lane evaluates one or two exponentials instead of CMAX.  The other classes' terms are summed
        // separately from the label's: near convergence softmax[label] is within an ulp of 1, and both the loss log(1 +
        // others / own) and the label's delta -(others / total) keep full relative accuracy this way, where log(total) -
        // logit and softmax - 1 would cancel.
        float logit[CT], ex[CT];
        float mx = -INFINITY;
#pragma unroll
        for (int c0 = 0; c0 < CT; ++c0) {
            float v = 0.0f;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) v += s_part[w][row * CMAX + kRow * c0 + sub];
            logit[c0] = kRow * c0 + sub < C ? v + bias[c0] : -INFINITY;
            mx = fmaxf(mx, logit[c0]);
        }
        mx = row_max(mx);
        float others = 0.0f, own = 0.0f, picked = 0.0f;
#pragma unroll
        for (int c0 = 0; c0 < CT; ++c0) {
            ex[c0] = expf(logit[c0] - mx);            // exp(-inf) = 0 for the padding
            const bool is_label = kRow * c0 + sub == label;
            own += is_label ? ex[c0] : 0.0f;
            picked += is_label ? logit[c0] : 0.0f;
            others += is_label ? 0.0f : ex[c0];
        }
        others = row_sum(others);
        own = row_sum(own);          // one non-zero term
        picked = row_sum(picked);    // one non-zero term
        const float sum = others + own;
        const float scale = 1.0f / (sum * (float)B);   // dlogits = (softmax - onehot) / B
        if (live && sub == 0)
            p.loss_parts[(int64_t)i * B + s] = own > 1e-30f ? log1pf(others / own) : (logf(sum) + mx) - picked;
#pragma unroll
        for (int c0 = 0; c0 < CT; ++c0) {
            const int c = kRow * c0 + sub;
            const float dv = (c == label ? -others : ex[c0]) * scale;   // 0 for the padding
            s_d[row][c] = dv;
            if (live && c < C) p.dlogits[((int64_t)i * B + s) * C + c] = dv;
        }
    }
    if (!p.dz) return;
    __syncthreads();
    // dz[s][k] = (sum_c dlogits[s][c] W[k][c]) * [h[s][k] > 0]
    float d[CS];
#pragma unroll
    for (int c = 0; c < CS; ++c) d[c] = s_d[l16][4 * c + q];
    const rsrc_t dz_rs = make_rsrc((char*)p.dz + ((int64_t)i * B * H + (int64_t)s0 * H) * es, (unsigned)rows * (unsigned)H * es);
#pragma unroll 1
    for (int c0 = 0; c0 < H; c0 += kChunk) {
        const int k0 = c0 + wave * T * 16;
        if (!one_pass) {
            load_h(k0);
            load_w2(k0);
        }
#pragma unroll
        for (int t = 0; t < T; ++t) {
            f4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < CS; ++c) o = __builtin_amdgcn_mfma_f32_16x16x4f32(w2[t][c], d[c], o, 0, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = h_elem(t, e) > 0.0f ? o[e] : 0.0f;
            const int k = k0 + 16 * t + 4 * q;
            const unsigned off = k < H ? ((unsigned)l16 * (unsigned)H + (unsigned)k) * es : kHeadNowhere;   // samples past the batch are dropped as well
            if constexpr (BF) {
                const u2 w = {f32_to_bf16(o[0]) | (f32_to_bf16(o[1]) << 16), f32_to_bf16(o[2]) | (f32_to_bf16(o[3]) << 16)};
                __builtin_amdgcn_raw_buffer_store_b64(w, dz_rs, (int)off, 0, 0);
            } else {
                buf_store(__builtin_bit_cast(u4, o), dz_rs, off);
            }
        }
    }
}

// Output-layer gradients as a kernel of their own (the body lives in head_dw_body.h, where it also serves as a
// guest of the weight-gradient GEMM's launch).  grid (ceil(H / 32), m)
template <bool BF, int CMAX>
__global__ __launch_bounds__(kHeadDwThreads) void head_dw_kernel(HeadDwDev a) {
    constexpr int kRows = CMAX > 16 ? 128 : 256;      // samples staged per pass (LDS stays below 64 KiB)
    __shared__ __attribute__((aligned(16))) float lds[head_dw_lds_floats(CMAX, kRows)];
    head_dw_body<BF, CMAX, kRows>(a, lds, blockIdx.x, blockIdx.y);
}

static bool head_args_ok(const HeadArgs& a) {
    return a.h && a.x && a.g && a.labels && a.dlogits && a.loss_parts && a.m >= 1 && a.m <= 65535 && a.B >= 1 &&
           a.H >= 4 && a.H % 4 == 0 && a.C >= 1 && a.C <= kMaxC && a.w_off >= 0 && a.b_off >= 0 &&
           a.w_off + (int64_t)a.H * a.C <= a.ld && a.b_off + a.C <= a.ld &&
           (reinterpret_cast<uintptr_t>(a.h) & 15u) == 0 && a.h_stride % 4 == 0;
}

template <bool BF, int CMAX, int T, int WAVES>
static hipError_t head_fwd_launch(const HeadDev& p, int m, hipStream_t s) {
    dim3 grid((unsigned)((p.B + 15) / 16), (unsigned)m);
    head_fwd_kernel<BF, CMAX, T, WAVES><<<grid, 64 * WAVES, 0, s>>>(p);
    return hipGetLastError();
}
// With partial sums to add up first, as many wavefronts as make that one item per lane (16 samples x H / 4 channel quads; wavefronts
// without units add zeros to the logits, the same bits).  One pass over the layer where the registers of up to 16 wavefronts hold it: T = 8 tiles of 16 units each, with fp32
// activations beyond 1024 units or with more than 16 classes four (eight spill).
template <bool BF>
static hipError_t head_fwd_dispatch(const HeadDev& p, int m, hipStream_t s) {
    const int units = p.pool.part ? 4 * p.H : p.H;
    if (p.C > 16) {
        if (units <= 256) return head_fwd_launch<BF, 32, 4, 4>(p, m, s);
        return head_fwd_launch<BF, 32, 4, 8>(p, m, s);
    }
    if (units <= 256) return head_fwd_launch<BF, 16, 4, 4>(p, m, s);
    if (units <= 512) return head_fwd_launch<BF, 16, 4, 8>(p, m, s);
    if (p.H <= 1024 && !p.pool.part) return head_fwd_launch<BF, 16, 8, 8>(p, m, s);
    if constexpr (BF) return head_fwd_launch<BF, 16, 8, 16>(p, m, s);
    return head_fwd_launch<BF, 16, 4, 16>(p, m, s);
}

// logits, loss, dlogits, and (when a.dz is set) the delta of the last hidden layer
hipError_t launch_head_fwd(const HeadArgs& a, hipStream_t s) {
    if (!head_args_ok(a)) return hipErrorInvalidValue;
    // 16-byte activation vectors: 4 floats or 8 bf16
    if (a.h_bf16 && (a.H % 8 || a.h_stride % 8)) return hipErrorInvalidValue;
    if (a.dz && (reinterpret_cast<uintptr_t>(a.dz) & 15u)) return hipErrorInvalidValue;
    if (a.pool.part && (a.h_bf16 || a.pool.per < 64 || (int64_t)a.B * a.pool.per >= ((int64_t)1 << 31) - 64 || a.pool.s_part % 4 ||
                        (reinterpret_cast<uintptr_t>(a.pool.part) & 15u) || (reinterpret_cast<uintptr_t>(a.pool.more) & 15u)))
        return hipErrorInvalidValue;
    HeadDev p;
    p.pool = a.pool;
    p.h = a.h;
    p.x = a.x;
    p.labels = a.labels;
    p.dlogits = a.dlogits;
    p.loss_parts = a.loss_parts;
    p.dz = a.dz;
    p.h_stride = a.h_stride;
    p.ld = a.ld;
    p.w_off = a.w_off;
    p.b_off = a.b_off;
    p.label_stride = a.label_stride;
    p.B = a.B;
    p.H = a.H;
    p.C = a.C;
    if (a.H >= (1 << 24)) return hipErrorInvalidValue;   // 32-bit byte offsets in the weights and in 16 samples' activations
    return a.h_bf16 ? head_fwd_dispatch<true>(p, a.m, s) : head_fwd_dispatch<false>(p, a.m, s);
}

// Validates the arguments of the output layer's gradient pass and lays them out for the device.
hipError_t head_dw_prepare(const HeadArgs& a, HeadDwDev* out) {
    if (!head_args_ok(a)) return hipErrorInvalidValue;
    if (a.upd.enabled && (!a.upd.x_in || !a.upd.x_out || (a.upd.mu != 0.0f && !a.upd.buf) || (a.upd.pull && !a.upd.z) ||
                          a.upd.ld != a.ld))
        return hipErrorInvalidValue;
    HeadDwDev d = {};
    d.h = a.h;
    d.dlogits = a.dlogits;
    d.g = a.g;
    d.h_stride = a.h_stride;
    d.ld = a.ld;
    d.w_off = a.w_off;
    d.b_off = a.b_off;
    d.B = a.B;
    d.H = a.H;
    d.C = a.C;
    d.bf16 = a.h_bf16 ? 1 : 0;
    d.grid_x = (a.H + kHeadDwUnits - 1) / kHeadDwUnits;
    const int64_t live = (int64_t)d.grid_x * a.m;
    if (live > (1 << 24)) return hipErrorInvalidValue;
    d.live = (int)live;
    d.blocks = (int)round_up(live, 8);   // a host launch keeps its own workgroup -> XCD assignment
    d.upd = a.upd;
    *out = d;
    return hipSuccess;
}

// gradients of the output layer's weights and bias (stored to g, or consumed by the fused update)
hipError_t launch_head_bwd(const HeadArgs& a, hipStream_t s) {
    HeadDwDev d;
    hipError_t e = head_dw_prepare(a, &d);
    if (e != hipSuccess) return e;
    dim3 grid((unsigned)d.grid_x, (unsigned)a.m);
    if (a.h_bf16) {
        if (a.C <= 16) head_dw_kernel<true, 16><<<grid, kHeadDwThreads, 0, s>>>(d);
        else head_dw_kernel<true, 32><<<grid, kHeadDwThreads, 0, s>>>(d);
    } else {
        if (a.C <= 16) head_dw_kernel<false, 16><<<grid, kHeadDwThreads, 0, s>>>(d);
        else head_dw_kernel<false, 32><<<grid, kHeadDwThreads, 0, s>>>(d);
    }
    return hipGetLastError();
}

}  // namespace ols
