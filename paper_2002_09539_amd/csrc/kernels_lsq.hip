// Per-worker stochastic gradient of the linear least-squares model: for worker i with mini-batch
// A [B][d], y [B] and parameters x^{(i)}:  r = A x - y,  loss = (1/B) sum_s 0.5 r_s^2,
// g = (1/B) A^T r  (the g_i(x; xi) of Section 2, arXiv 2002.09539, for this model).
// The problem is tiny (B x d = 32 x 1024 per worker) and latency-bound; plain vector ALU code.
#include <atomic>
#include <type_traits>

#include "ols_internal.h"

namespace ols {

constexpr int kThreads = 256;

// one workgroup per (sample s, worker i): r[i][s] = A[i][s][:] . x[i][:] - y[i][s]
__global__ __launch_bounds__(kThreads) void lsq_resid_kernel(const float* __restrict__ A, int64_t a_stride,
                                                             const float* __restrict__ y, int64_t y_stride,
                                                             const float* __restrict__ x, int64_t ld,
                                                             float* __restrict__ resid, float* __restrict__ loss_parts,
                                                             int B, int64_t d) {
    const int s = blockIdx.x, i = blockIdx.y;
    const float* row = A + (int64_t)i * a_stride + (int64_t)s * d;
    const float* xi = x + (int64_t)i * ld;
    float acc = 0.0f;
    for (int64_t j = threadIdx.x; j < d; j += kThreads) acc = __fmaf_rn(row[j], xi[j], acc);
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    __shared__ float part[kThreads / 64];
    if (threadIdx.x % 64 == 0) part[threadIdx.x / 64] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        float r = 0.0f;
        for (int w = 0; w < kThreads / 64; ++w) r += part[w];
        r -= y[(int64_t)i * y_stride + s];
        resid[(int64_t)i * B + s] = r;
        loss_parts[(int64_t)i * B + s] = 0.5f * r * r;
    }
}

// one lane per parameter j of worker i: g[i][j] = (1/B) sum_s A[i][s][j] r[i][s]
__global__ __launch_bounds__(kThreads) void lsq_grad_kernel(const float* __restrict__ A, int64_t a_stride,
                                                            const float* __restrict__ resid, float* __restrict__ g,
                                                            int64_t ld, int B, int64_t d) {
    extern __shared__ float r_lds[];
    const int i = blockIdx.y;
    for (int s = threadIdx.x; s < B; s += kThreads) r_lds[s] = resid[(int64_t)i * B + s];
    __syncthreads();
    const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (j >= d) return;
    const float* col = A + (int64_t)i * a_stride + j;
    float acc = 0.0f;
#pragma unroll 16   // independent loads ahead of the dependent chain of additions
    for (int s = 0; s < B; ++s) acc = __fmaf_rn(col[(int64_t)s * d], r_lds[s], acc);
    g[(int64_t)i * ld + j] = acc / (float)B;
}

// Small problems: residuals, loss, gradient and the local step (+ pull-back) of a worker by one workgroup of 1024 threads,
// for one step or for all the steps up to a synchronisation -- a worker's local steps read nothing of the others', so
// parameters and momenta stay in registers between them -- and, with the round's last step, the anchor as well: the
// workgroup that finishes last averages the replicas (replica by replica in the order of mean_kernel, identical bits).
//
// What bounds it is latency: 131 kFLOP and 128 KiB of data per worker and step, and every instruction is fetched for a
// handful of uses, so each case is compiled for itself (one step or several, up to 32 samples or more).  Measured on 4
// workers x 1024 parameters, batch 32, tau = 2, us per round, one after the other: a launch per step and one for the mean 17.3;
// the round in one launch 11.0 with the code of all cases in one kernel and the average's partial sums in scratch memory,
// now 9.3.  With a copy of the mini-batch in LDS between residuals and gradient and three agent-wide fences by every
// thread it took 24.
//
// How the last workgroup is known without a counter that somebody has to clear: every launch carries a stamp that no
// launch before it had; a workgroup publishes its replica, writes the stamp into its own flag and then reads all flags.
// The one that finds m stamps is the last (or one of several that finished together: they write the same values).  It
// clears the flags, after which no workgroup writes one; whoever reads them then leaves the average to it.
typedef float lsq_f4 __attribute__((ext_vector_type(4)));
constexpr int kStepThreads = 1024, kStepMaxB = 64, kStepMaxCols = 4;

struct LsqRound {
    const float* A;          // first batch of worker 0
    const float* y;
    int64_t a_stride, y_stride, a_batch, y_batch;   // elements between workers and between batches
    float* loss_parts;       // of the last step
    int B, d, nb, first_batch, steps, m;
    FusedUpdate u;           // u.pull: the last step is followed by the pull-back
    unsigned long long* flags;   // [m] with mean, else unused
    unsigned long long stamp;
    float* z;                // with mean: the anchor
    int mean, mean_split;
};

// The average of one column over the replicas as mean_kernel<..., SW, SL> forms it: group f of G = SW * SL adds rows f, f + G,
// ... in order, lane groups combine by exchange, wavefront groups by a tree.
template <int G>
__device__ __forceinline__ float lsq_column_mean(const float* x, int64_t ld, int j, int m) {
    constexpr int SW = G < 4 ? G : 4, SL = G / SW;
    float part[G];
#pragma unroll
    for (int f = 0; f < G; ++f) part[f] = 0.0f;
    for (int i = 0; i < m; i += G) {   // (the split that the mean kernel chooses leaves one or two passes)
        float v[G];
#pragma unroll
        for (int f = 0; f < G; ++f) v[f] = __hip_atomic_load(x + (int64_t)min(i + f, m - 1) * ld + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int f = 0; f < G; ++f)
            if (i + f < m) part[f] = __fadd_rn(part[f], v[f]);
    }
#pragma unroll
    for (int w = 0; w < SW; ++w)
#pragma unroll
        for (int off = 1; off < SL; off <<= 1)
#pragma unroll
            for (int l = 0; l < SL; l += 2 * off) part[w * SL + l] = __fadd_rn(part[w * SL + l], part[w * SL + l + off]);
#pragma unroll
    for (int stride = SW / 2; stride >= 1; stride >>= 1)
#pragma unroll
        for (int w = 0; w < stride; ++w) part[w * SL] = __fadd_rn(part[w * SL], part[(w + stride) * SL]);
    return anchor_mean_elem(part[0], (float)m);
}

// Behind the round's last step: publishes this workgroup's replica, and the workgroup that finds itself last averages all
// of them.  A workgroup barrier does not wait for vector stores, so every wavefront first waits until its own have reached
// the XCD's L2; one release (the write-back of that L2) per workgroup follows.  The exchange has taken effect when it
// returns, so of two workgroups at least the later one reads both flags.
__device__ void lsq_round_mean(const LsqRound& p, int i, int t) {
    const FusedUpdate& u = p.u;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (t == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        (void)__hip_atomic_exchange(p.flags + i, p.stamp, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    bool all = true;
    for (int k = t; k < p.m; k += kStepThreads) all = all && __hip_atomic_load(p.flags + k, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) == p.stamp;
    if (!__syncthreads_and(all)) return;
    auto columns = [&](auto groups) {
        for (int j = t; j < p.d; j += kStepThreads) p.z[j] = lsq_column_mean<decltype(groups)::value>(u.x_out, u.ld, j, p.m);
    };
    switch (p.mean_split) {
        case 1: columns(std::integral_constant<int, 1>{}); break;
        case 2: columns(std::integral_constant<int, 2>{}); break;
        case 4: columns(std::integral_constant<int, 4>{}); break;
        case 8: columns(std::integral_constant<int, 8>{}); break;
        default: columns(std::integral_constant<int, 16>{}); break;
    }
    // every flag has been written for this launch: leave none of its stamps behind (a captured launch carries its stamp
    // into every replay)
    for (int k = t; k < p.m; k += kStepThreads) __hip_atomic_store(p.flags + k, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum over the 64 lanes, in every lane: within rows of 16 lanes by exchanges between neighbours, then the four rows.
__device__ __forceinline__ float wave_sum(float v) {
    auto add = [&](auto ctrl) {
        v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xF, 0xF, true));
    };
    add(std::integral_constant<int, 0xB1>{});    // lane ^ 1
    add(std::integral_constant<int, 0x4E>{});    // lane ^ 2
    add(std::integral_constant<int, 0x141>{});   // mirrored within 8
    add(std::integral_constant<int, 0x140>{});   // mirrored within 16
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
    return (r0 + r1) + (r2 + r3);
}

// At most 1024 columns, a multiple of four.  A wavefront takes two samples at a time and holds their rows in registers:
// dot products, residuals and the two samples' share of the gradient come from one read; the shares of the sixteen
// wavefronts meet in LDS.  With at most 32 samples the next step's rows are on their way meanwhile.
template <bool ROUNDS, bool PASSES>
__global__ __launch_bounds__(kStepThreads) void lsq_round_narrow_kernel(LsqRound p) {
    constexpr int kWaves = kStepThreads / 64, kRows = 2, kCols = 1024;
    __shared__ lsq_f4 s_x[kCols / 4];
    __shared__ lsq_f4 s_p[kWaves][kCols / 4];
    const FusedUpdate& u = p.u;
    const int i = blockIdx.x, t = threadIdx.x, B = p.B, d = p.d;
    const int wave = t / 64, lane = t % 64;
    const bool mom = u.mu != 0.0f, own = t < d;
    const int64_t at = (int64_t)i * u.ld + t;
    const float* A0 = p.A + (int64_t)i * p.a_stride;
    const float* y0 = p.y + (int64_t)i * p.y_stride;
    lsq_f4 a[kRows][4];
    float yv[kRows];
    auto load_rows = [&](int batch, int s0) {
        const float* Ai = A0 + batch * p.a_batch;
        const float* yi = y0 + batch * p.y_batch;
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int s = s0 + r * kWaves;
            yv[r] = s < B ? yi[s] : 0.0f;
            const lsq_f4* row = (const lsq_f4*)(Ai + (int64_t)(s < B ? s : 0) * d) + lane;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool ok = s < B && 4 * (lane + 64 * e) < d;
                const lsq_f4 v = row[ok ? 64 * e : -lane];   // out of range: the row's first vector, not used
                a[r][e] = ok ? v : lsq_f4{0.f, 0.f, 0.f, 0.f};
            }
        }
    };
    int batch = p.first_batch;
    float x = own ? u.x_in[at] : 0.0f;
    float b = own && mom ? u.buf[at] : 0.0f;
    const float z = own && u.pull ? u.z[t] : 0.0f;
    load_rows(batch, wave);
    ((float*)s_x)[t] = x;
    __syncthreads();
    const float fB = (float)B;
    const int steps = ROUNDS ? p.steps : 1;
    for (int st = 0; st < steps; ++st) {
        const bool last = st + 1 == steps;
        const int next = batch + 1 < p.nb ? batch + 1 : 0;
        lsq_f4 g[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) g[e] = lsq_f4{0.f, 0.f, 0.f, 0.f};
        for (int s0 = wave; s0 < B; s0 += kRows * kWaves) {
            if (PASSES && s0 != wave) load_rows(batch, s0);
            lsq_f4 dot[kRows];
#pragma unroll
            for (int r = 0; r < kRows; ++r) dot[r] = lsq_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const lsq_f4 xe = s_x[lane + 64 * e];
#pragma unroll
                for (int r = 0; r < kRows; ++r)
#pragma unroll
                    for (int k = 0; k < 4; ++k) dot[r][k] = __fmaf_rn(a[r][e][k], xe[k], dot[r][k]);
            }
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                const int s = s0 + r * kWaves;
                const float res = wave_sum((dot[r][0] + dot[r][1]) + (dot[r][2] + dot[r][3])) - yv[r];
                if (last && lane == 0 && s < B) p.loss_parts[(int64_t)i * B + s] = 0.5f * res * res;
                if (s < B) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int k = 0; k < 4; ++k) g[e][k] = __fmaf_rn(a[r][e][k], res, g[e][k]);
                }
            }
            if (!PASSES) break;
        }
        // what the next step reads first: its first two rows per wavefront
        if (!last) load_rows(next, wave);
        batch = next;
#pragma unroll
        for (int e = 0; e < 4; ++e) s_p[wave][lane + 64 * e] = g[e];
        __syncthreads();
        float sum = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) sum += ((const float*)s_p[w])[t];
        x = local_step_elem(sum / fB, x, b, z, u.gamma, u.mu, u.alpha, mom, u.nesterov != 0, u.pull != 0 && last);
        if (!last) {
            ((float*)s_x)[t] = own ? x : 0.0f;
            __syncthreads();
        }
    }
    if (own) {
        if (mom) u.buf[at] = b;
        u.x_out[at] = x;
    }
    if (p.mean) lsq_round_mean(p, i, t);
}

// More columns, or a number that is no multiple of four: rows in passes of 1024 columns, the gradient from a second read.
__global__ __launch_bounds__(kStepThreads) void lsq_round_wide_kernel(LsqRound p) {
    constexpr int kWaves = kStepThreads / 64, kRows = 2, kFly = 16;
    __shared__ float s_x[kStepMaxCols * kStepThreads];     // parameters
    __shared__ float s_r[kStepMaxB];                       // residuals
    const FusedUpdate& u = p.u;
    const int i = blockIdx.x, t = threadIdx.x, B = p.B, d = p.d;
    const int wave = t / 64, lane = t % 64;
    const bool mom = u.mu != 0.0f;
    float xv[kStepMaxCols], bv[kStepMaxCols], zv[kStepMaxCols];
#pragma unroll
    for (int c = 0; c < kStepMaxCols; ++c) {
        const int j = t + c * kStepThreads;
        const bool ok = j < d;
        xv[c] = ok ? u.x_in[(int64_t)i * u.ld + j] : 0.0f;
        bv[c] = (ok && mom) ? u.buf[(int64_t)i * u.ld + j] : 0.0f;
        zv[c] = (ok && u.pull) ? u.z[j] : 0.0f;
        if (ok) s_x[j] = xv[c];
    }
    const float* A0 = p.A + (int64_t)i * p.a_stride;
    const float* y0 = p.y + (int64_t)i * p.y_stride;
    int batch = p.first_batch;
    __syncthreads();
    for (int st = 0; st < p.steps; ++st) {
        const bool last = st + 1 == p.steps;
        const float* Ai = A0 + batch * p.a_batch;
        const float* yi = y0 + batch * p.y_batch;
        batch = batch + 1 < p.nb ? batch + 1 : 0;
        for (int s0 = wave; s0 < B; s0 += kRows * kWaves) {
            float acc[kRows] = {0.0f, 0.0f};
            for (int c0 = 0; c0 < d; c0 += kFly * 64) {
                float a[kRows][kFly];
#pragma unroll
                for (int r = 0; r < kRows; ++r) {   // all loads of the pass before their first use
                    const int s = s0 + r * kWaves;
                    const float* row = Ai + (int64_t)(s < B ? s : 0) * d;
#pragma unroll
                    for (int e = 0; e < kFly; ++e) {
                        const int j = c0 + lane + 64 * e;
                        a[r][e] = row[j < d ? j : 0];
                    }
                }
#pragma unroll
                for (int e = 0; e < kFly; ++e) {
                    const int j = c0 + lane + 64 * e;
                    if (j < d) {
                        const float xj = s_x[j];
#pragma unroll
                        for (int r = 0; r < kRows; ++r) acc[r] = __fmaf_rn(a[r][e], xj, acc[r]);
                    }
                }
            }
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                const int s = s0 + r * kWaves;
                const float dot = wave_sum(acc[r]);
                if (lane == 0 && s < B) {
                    const float res = dot - yi[s];
                    s_r[s] = res;
                    if (last) p.loss_parts[(int64_t)i * B + s] = 0.5f * res * res;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kStepMaxCols; ++c) {
            const int j = t + c * kStepThreads;
            if (j >= d) break;
            float g = 0.0f;
#pragma unroll 8
            for (int s = 0; s < B; ++s) g = __fmaf_rn(Ai[(int64_t)s * d + j], s_r[s], g);
            xv[c] = local_step_elem(g / (float)B, xv[c], bv[c], zv[c], u.gamma, u.mu, u.alpha, mom, u.nesterov != 0, u.pull != 0 && last);
            if (!last) s_x[j] = xv[c];
        }
        if (!last) __syncthreads();
    }
#pragma unroll
    for (int c = 0; c < kStepMaxCols; ++c) {
        const int j = t + c * kStepThreads;
        if (j >= d) break;
        if (mom) u.buf[(int64_t)i * u.ld + j] = bv[c];
        u.x_out[(int64_t)i * u.ld + j] = xv[c];
    }
    if (p.mean) lsq_round_mean(p, i, t);
}

// One step of such a problem while the mini-batch is small: a launch this short pays for every instruction it fetches, so the
// loops are short and rolled.  The sums are those of lsq_round_wide_kernel, in the same order: identical bits.
__global__ __launch_bounds__(kStepThreads) void lsq_step_kernel(LsqRound p) {
    constexpr int kWaves = kStepThreads / 64;
    __shared__ float s_r[kStepMaxB];
    const FusedUpdate& u = p.u;
    const int i = blockIdx.x, t = threadIdx.x, B = p.B, d = p.d;
    const int wave = t / 64, lane = t % 64;
    const bool mom = u.mu != 0.0f;
    const float* Ai = p.A + (int64_t)i * p.a_stride + p.first_batch * p.a_batch;
    const float* yi = p.y + (int64_t)i * p.y_stride + p.first_batch * p.y_batch;
    const float* xi = u.x_in + (int64_t)i * u.ld;
    float xv[kStepMaxCols], bv[kStepMaxCols], zv[kStepMaxCols];
#pragma unroll
    for (int c = 0; c < kStepMaxCols; ++c) {
        const int j = t + c * kStepThreads;
        const bool ok = j < d;
        xv[c] = ok ? xi[j] : 0.0f;
        bv[c] = (ok && mom) ? u.buf[(int64_t)i * u.ld + j] : 0.0f;
        zv[c] = (ok && u.pull) ? u.z[j] : 0.0f;
    }
    for (int s = wave; s < B; s += kWaves) {
        const float* row = Ai + (int64_t)s * d;
        float acc = 0.0f;
#pragma unroll 4
        for (int j = lane; j < d; j += 64) acc = __fmaf_rn(row[j], xi[j], acc);
        const float dot = wave_sum(acc);
        if (lane == 0) {
            const float res = dot - yi[s];
            s_r[s] = res;
            p.loss_parts[(int64_t)i * B + s] = 0.5f * res * res;
        }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kStepMaxCols; ++c) {
        const int j = t + c * kStepThreads;
        if (j >= d) break;
        float g = 0.0f;
#pragma unroll 8
        for (int s = 0; s < B; ++s) g = __fmaf_rn(Ai[(int64_t)s * d + j], s_r[s], g);
        fused_update_store(u, (int64_t)i * u.ld + j, g / (float)B, xv[c], bv[c], zv[c]);
    }
}

bool lsq_step_fits(int B, int64_t d) { return B >= 1 && B <= kStepMaxB && d >= 1 && d <= kStepMaxCols * kStepThreads; }

static bool narrow_columns(int64_t d) { return d <= 1024 && d % 4 == 0; }
// whether the wide kernel's passes of 32 samples x 1024 columns are filled to at least `percent`
static bool wide_fill(int B, int64_t d, int percent) {
    return 100 * B * d >= (int64_t)percent * round_up(B, 32) * round_up(d, 1024);
}

// The rules, from 2 .. 64 workers x 64 .. 4096 columns x 4 .. 64 samples with tau 1, 2 and 4 (us per round; the other side is
// a launch per step and one for the average):
// - The narrow kernel is as fast or faster (4 x 256 x 8, tau 2: 8.0 against 11.7; 64 x 64 x 64, tau 2, 17.0 against 16.2 is
//   the worst), and so are whole rounds of ragged rows up to 1024 columns (8 x 201 x 8, tau 2: 8.7 against 11.0).
// - The wide kernel's passes cost the same empty or full.  Whole rounds from half full on with more than 16 samples: 2 x 1500 x
//   24, tau 2, 15.5 against 17.7, 2 x 2048 x 24 18.4 against 19.5; below, 2 x 4096 x 8 21.2 against 17.3, 2 x 1028 x 48 21.5
//   against 20.6.  With fewer samples and up to 1536 columns what the launches cost decides: rounds of three steps on, or of
//   two with their average (2 x 1500 x 8, tau 4: 9 % faster, tau 2 even).
// - Single steps take the wide kernel where its samples fill whole passes (two of 2 x 2500 x 32 and the average 25.1 against
//   27.0 with the kernel for one step; of 2 x 2048 x 24 21.1 against 19.4).
// - The last workgroup averages up to 64 KiB from at most 32 replicas of at most 2048 columns (32 x 256 x 8, tau 1: 7.6
//   against 10.2; 64 x 256 x 8 9.6 and 9.7; 2 x 2048 x 32, tau 2, 18.9 against 22.0; 2 x 3000 x 4 19.1 and 17.9); more is left
//   to the mean kernel's many workgroups.
bool lsq_round_pays(int B, int64_t d, int64_t steps, bool with_mean) {
    if (d <= 1024 || (B > 16 && wide_fill(B, d, 50))) return true;
    return d <= 1536 && (steps >= 3 || (steps == 2 && with_mean));
}

bool lsq_round_with_mean(int m, int64_t d, int64_t ld) { return m <= 32 && d <= 2048 && m * ld <= 16384; }

hipError_t launch_lsq_round(const LsqRoundArgs& a, const FusedUpdate& u, hipStream_t s) {
    if (!a.A || !a.y || !a.loss_parts || a.m < 1 || !lsq_step_fits(a.B, a.d) || a.nb < 1 || a.first_batch < 0 || a.first_batch >= a.nb ||
        a.steps < 1 || !u.enabled || !u.x_in || !u.x_out || u.ld < a.d || (u.mu != 0.0f && !u.buf) || (u.pull && !u.z) || u.shadow)
        return hipErrorInvalidValue;
    if (a.with_mean && (!u.pull || !a.flags || !a.z || !lsq_round_with_mean(a.m, a.d, u.ld))) return hipErrorInvalidValue;
    static std::atomic<unsigned long long> launches{0};   // stamps only have to differ from launch to launch
    LsqRound p = {};
    p.A = a.A; p.y = a.y;
    p.a_stride = a.a_stride; p.y_stride = a.y_stride; p.a_batch = (int64_t)a.B * a.d; p.y_batch = a.B;
    p.loss_parts = a.loss_parts;
    p.B = a.B; p.d = (int)a.d; p.nb = a.nb; p.first_batch = a.first_batch; p.steps = a.steps; p.m = a.m;
    p.u = u;
    p.flags = a.flags;
    p.z = a.z;
    p.mean = a.with_mean ? 1 : 0;
    if (p.mean) {
        p.stamp = ++launches * 0x9E3779B97F4A7C15ull;   // no small integer that stale memory might hold
        p.mean_split = a.mean_split > 0 ? a.mean_split : mean_auto_split(a.m, u.ld);
    }
    if (narrow_columns(a.d) && !(reinterpret_cast<uintptr_t>(a.A) & 15u) && a.a_stride % 4 == 0) {
        auto kern = a.B > 32 ? (a.steps > 1 ? lsq_round_narrow_kernel<true, true> : lsq_round_narrow_kernel<false, true>)
                             : (a.steps > 1 ? lsq_round_narrow_kernel<true, false> : lsq_round_narrow_kernel<false, false>);
        kern<<<(unsigned)a.m, kStepThreads, 0, s>>>(p);
        return hipGetLastError();
    }
    const bool filled = wide_fill(a.B, a.d, 70) && round_up(a.B, 32) - a.B < 4;
    if (a.steps == 1 && !p.mean && !filled) lsq_step_kernel<<<(unsigned)a.m, kStepThreads, 0, s>>>(p);
    else lsq_round_wide_kernel<<<(unsigned)a.m, kStepThreads, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_lsq_resid(const float* A, int64_t a_stride, const float* y, int64_t y_stride, const float* x,
                            int64_t ld, float* resid, float* loss_parts, int m, int B, int64_t d, hipStream_t s) {
    if (!A || !y || !x || !resid || !loss_parts || m < 1 || m > 65535 || B < 1 || d < 1 || ld < d)
        return hipErrorInvalidValue;
    lsq_resid_kernel<<<dim3((unsigned)B, (unsigned)m), kThreads, 0, s>>>(A, a_stride, y, y_stride, x, ld, resid,
                                                                        loss_parts, B, d);
    return hipGetLastError();
}

hipError_t launch_lsq_grad(const float* A, int64_t a_stride, const float* resid, float* g, int64_t ld, int m, int B,
                           int64_t d, hipStream_t s) {
    if (!A || !resid || !g || m < 1 || m > 65535 || B < 1 || B > 8192 || d < 1 || ld < d) return hipErrorInvalidValue;
    dim3 grid((unsigned)((d + kThreads - 1) / kThreads), (unsigned)m);
    lsq_grad_kernel<<<grid, kThreads, (size_t)B * sizeof(float), s>>>(A, a_stride, resid, g, ld, B, d);
    return hipGetLastError();
}

}  // namespace ols
