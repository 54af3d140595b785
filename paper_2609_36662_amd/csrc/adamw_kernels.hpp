// Inner AdamW step of K workers on gfx950 (the local inner loops between two
// synchronisations; settings of Table "Training settings": AdamW with
// coefficients (beta1, beta2), weight decay, gradient-norm clipping; App. G.1:
// FP32 master parameters and AdamW states, BF16 compute copy).
//
// Two streaming passes, both bound by HBM bandwidth:
//   grad_norm_kernel  reads every worker's gradient once and sums g^2 per
//                     worker (fp32 per vector, fp64 per lane, then the same
//                     deterministic two-stage reduction as the round), so the
//                     clipping coefficient sees the worker's whole gradient;
//   adamw_kernel      one grid row per worker: reads theta, m, v and g once,
//                     writes theta, m, v once (and the BF16 copy of theta):
//                       c      = min(1, max_norm / (||g|| + 1e-6))   (from pass 1)
//                       g      = c g
//                       theta  = theta (1 - lr wd)
//                       m      = beta1 m + (1 - beta1) g
//                       v      = beta2 v + (1 - beta2) g^2
//                       theta -= (lr / (1 - beta1^t)) m / (sqrt(v) / sqrt(1 - beta2^t) + eps)
// The clipping coefficient is computed in fp64 by every workgroup of pass 2 from
// the per-workgroup sums pass 1 left in device memory, so the step needs neither a
// host round trip nor a kernel between the passes.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "reduce.hpp"
#include "round_kernels.hpp"

namespace autoloco {

struct GradNormArgs {
    const float* grads[kMaxK];
    int64_t n;
    double* partials;      // [K][gridDim.x] per-workgroup squared norms
};

struct AdamWArgs {
    float* params[kMaxK];
    float* exp_avg[kMaxK];
    float* exp_avg_sq[kMaxK];
    const float* grads[kMaxK];
    uint16_t* copy[kMaxK];   // BF16 copies of the new parameters, or all null
    int64_t n;
    const double* partials;  // [K][nblocks] per-workgroup squared norms, or null (no norms)
    int nblocks;
    double max_norm;         // 0: no clipping
    double* sums;            // [K] squared norms, written by each worker's first workgroup
    double* host_sums;       // the same in coherent host memory, or null
    float decay;             // 1 - lr * weight_decay
    float beta1, beta2;
    float omb1, omb2;        // 1 - beta1, 1 - beta2
    float step_size;         // lr / (1 - beta1^t)
    float inv_sqrt_bc2;      // 1 / sqrt(1 - beta2^t)
    float eps;
    uint32_t mask;           // traffic reference only: 0 (a value the compiler cannot see)
};

// Windows of its grid-stride sequence a thread loads before it adds any of them
// up (in that order, so every per-thread sum is what one window at a time gives):
// one worker's stream alone keeps too few bytes in flight at three workgroups a CU.
// (124M: K = 1 77 us against 109; from K = 3 on nothing is gained.)  The loads of a
// window of all workers go out together: left alone, the compiler puts more and more
// of them behind the first sums from K = 11 on, one at a time at K = 16 (whole step,
// 124M: K = 16 11.8 ms against 12.5, K = 15 11.1 against 11.7; 10,000 parameters
// 13.2 us against 18.9 and 17.0).
template <int K>
constexpr int norm_unroll() {
    return K == 1 ? 4 : K == 2 ? 2 : 1;
}

template <int K>
__global__ void __launch_bounds__(kBlock) grad_norm_kernel(GradNormArgs a) {
    constexpr int U = norm_unroll<K>();
    double acc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] = 0.0;
    const int64_t nvec = a.n / 4;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    auto add = [&](int k, f32x4 g) {
        float s = g[0] * g[0];
        s = __builtin_fmaf(g[1], g[1], s);
        s = __builtin_fmaf(g[2], g[2], s);
        s = __builtin_fmaf(g[3], g[3], s);
        acc[k] += (double)s;
    };
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if constexpr (U > 1) {
        for (; i + (U - 1) * stride < nvec; i += U * stride) {
            f32x4 g[U][K];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int k = 0; k < K; ++k) g[u][k] = ld_f4(a.grads[k] + 4 * (i + u * stride));
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int k = 0; k < K; ++k) add(k, g[u][k]);
        }
    }
    for (; i < nvec; i += stride) {
        f32x4 g[K];
#pragma unroll
        for (int k = 0; k < K; ++k) g[k] = ld_f4(a.grads[k] + 4 * i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < K; ++k) add(k, g[k]);
    }
    if (blockIdx.x == 0 && threadIdx.x < (a.n & 3)) {
        const int64_t j = nvec * 4 + threadIdx.x;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const float g = a.grads[k][j];
            acc[k] += (double)(g * g);
        }
    }
    store_partials<K, kBlock>(acc, a.partials);
}

// Clipping coefficient from a squared norm; NaN stays NaN.
__device__ __forceinline__ float clip_coef(double norm_sq, double max_norm) {
    const double c = max_norm / (sqrt(norm_sq) + 1e-6);
    return (float)(c > 1.0 ? 1.0 : c);
}

__device__ __forceinline__ void adamw_one(const AdamWArgs& a, float coef, float& p, float& m, float& v, float g) {
    g *= coef;
    const float pd = p * a.decay;
    m = __builtin_fmaf(a.beta1, m, a.omb1 * g);
    v = __builtin_fmaf(a.beta2, v, (a.omb2 * g) * g);
    const float denom = __builtin_fmaf(__builtin_sqrtf(v), a.inv_sqrt_bc2, a.eps);
    p = pd - a.step_size * (m / denom);
}

typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));

// One element of the traffic reference: the loaded words go back unchanged
// (a.mask is 0), and the gradient word is folded into the parameter's through
// the same mask so that its load stays.
__device__ __forceinline__ void adamw_keep(const AdamWArgs& a, float& p, float& m, float& v, float g) {
    p = __uint_as_float(__float_as_uint(p) ^ (__float_as_uint(g) & a.mask));
    m = __uint_as_float(__float_as_uint(m) ^ a.mask);
    v = __uint_as_float(__float_as_uint(v) ^ a.mask);
}

// TRAFFIC: the traffic reference of this kernel -- the same grid, loop, loads and
// stores, none of the arithmetic; θ, m and v keep their bits and the BF16 copy
// receives the rounding of the unchanged θ (what the last step wrote there).
template <bool COPY, bool TRAFFIC>
__global__ void __launch_bounds__(kBlock) adamw_kernel(AdamWArgs a) {
    const int k = blockIdx.y;
    float coef = 1.0f;
    if (!TRAFFIC && a.partials != nullptr) {
        // worker k's squared norm, added up in the order of the reductions' second
        // stage by every workgroup (a few KB from the caches), instead of in a
        // kernel between the passes
        __shared__ double total;
        double t[1] = {0.0};
        for (int b = threadIdx.x; b < a.nblocks; b += kBlock) t[0] += a.partials[(int64_t)k * a.nblocks + b];
        const double sum = block_reduce<1, kBlock>(t);
        if (threadIdx.x == 0) {
            total = sum;
            if (blockIdx.x == 0) {
                a.sums[k] = sum;
                if (a.host_sums != nullptr) a.host_sums[k] = sum;
            }
        }
        __syncthreads();
        if (a.max_norm > 0.0) coef = clip_coef(total, a.max_norm);
    }
    float* __restrict__ p = a.params[k];
    float* __restrict__ m = a.exp_avg[k];
    float* __restrict__ v = a.exp_avg_sq[k];
    const float* __restrict__ g = a.grads[k];
    uint16_t* __restrict__ c = a.copy[k];
    const int64_t nvec = a.n / 4;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    struct Quad {
        f32x4 p, m, v, g;
    };
    auto load = [&](int64_t i) { return Quad{ld_f4(p + 4 * i), ld_f4(m + 4 * i), ld_f4(v + 4 * i), ld_f4(g + 4 * i)}; };
    auto step = [&](int64_t i, const Quad& x) {
        float pe[4], me[4], ve[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            pe[e] = x.p[e];
            me[e] = x.m[e];
            ve[e] = x.v[e];
            if constexpr (TRAFFIC)
                adamw_keep(a, pe[e], me[e], ve[e], x.g[e]);
            else
                adamw_one(a, coef, pe[e], me[e], ve[e], x.g[e]);
        }
        st_f4(p + 4 * i, f32x4{pe[0], pe[1], pe[2], pe[3]});
        st_f4(m + 4 * i, f32x4{me[0], me[1], me[2], me[3]});
        st_f4(v + 4 * i, f32x4{ve[0], ve[1], ve[2], ve[3]});
        if constexpr (COPY)
            __builtin_nontemporal_store(u32x2v{bf16_pack(pe[0], pe[1]), bf16_pack(pe[2], pe[3])},
                                        reinterpret_cast<u32x2v*>(c + 4 * i));
    };
    // From the last window down: the norm pass read the gradients up to their ends
    // just before, and what the Infinity Cache still holds of them comes first.
    // (124M, K = 4: 2.57 ms against 2.60.)
    const int64_t nw = (nvec + kBlock - 1) / kBlock;
    int64_t i = (nw - 1 - blockIdx.x) * kBlock + threadIdx.x;
    if (blockIdx.x == 0) {   // the last window may be short, or missing (n < 4)
        if (i >= 0 && i < nvec) step(i, load(i));
        i -= stride;
    }
    // Many windows a workgroup: the next one is loaded before this one is worked on
    // (one workgroup a CU, update pass: 124M K = 4 2.45 ms against 2.53 without, K = 8
    // 5.01 against 5.15; on buffers spread in HBM 2.26 against 2.30 and 4.55 against
    // 4.65; whole step on the same buffers 1-5 % at every K from 30M to 200M).  Not with
    // few, where it gains nothing (1M, K = 4: 24.8 us against 24.2).  The loop's waits
    // cover the stores of the window before; two windows in turn, whose waits do not, are
    // slower (30M: K = 4 753 us against 644, K = 8 1.44 ms against 1.28; 124M K = 4 2.81
    // ms against 2.65): with more in flight the memory runs worse.
    if (nw >= 16 * (int64_t)gridDim.x && i >= 0) {
        Quad x = load(i);
        for (; i >= stride; i -= stride) {
            const Quad next = load(i - stride);
            __builtin_amdgcn_sched_barrier(0);
            step(i, x);
            x = next;
        }
        step(i, x);
    } else {
        for (; i >= 0; i -= stride) step(i, load(i));
    }
    if (blockIdx.x == 0 && threadIdx.x < (a.n & 3)) {
        const int64_t j = nvec * 4 + threadIdx.x;
        float pe = p[j], me = m[j], ve = v[j];
        if constexpr (TRAFFIC)
            adamw_keep(a, pe, me, ve, g[j]);
        else
            adamw_one(a, coef, pe, me, ve, g[j]);
        p[j] = pe;
        m[j] = me;
        v[j] = ve;
        if constexpr (COPY) c[j] = (uint16_t)bf16_rne(pe);
    }
}

hipError_t launch_grad_norm(int k, int blocks, hipStream_t s, const GradNormArgs& a);
hipError_t launch_adamw(bool copy, bool traffic, int k, int blocks_per_worker, hipStream_t s, const AdamWArgs& a);

}  // namespace autoloco
