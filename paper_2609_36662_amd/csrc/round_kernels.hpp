// Streaming kernels of one AutoLoCo synchronisation round on gfx950.
//
// One pass over the parameters reads theta_t, v_{t-1} and the K worker
// replicas once, and (depending on the mode) writes theta_{t+1}, v_t and the
// K reset replicas once.  Per parameter j:
//   Delta_k   = theta[j] - theta_k[j]                  (Alg. "AutoLoCo outer interval")
//   Delta_bar = (sum_k Delta_k) * (1/K)                pairwise tree over k in index order
//   S_k += Delta_k^2, Q_k += (Delta_k - Delta_bar)^2, M += Delta_bar^2
//                                                      (eq. adaptive-h-core-diagnostics; App. C.1)
//   Dt = Delta_bar * scale   (scale = 1/rho when normalising, else 1; eq. normalized-pseudo-gradient)
//   v' = mu v + Dt; d = Dt + mu v'; theta' = theta - eta d   (eq. autoloco-corrected-nesterov)
//   theta_k[j] = theta'  (fp32, or bf16 rounded to nearest even)
//
// Nothing here is a contraction, so no matrix cores are used: the work is
// bound by HBM bandwidth.  Each lane moves 16-byte vectors (4 fp32 or 8 bf16
// parameters) with non-temporal loads and stores so the streams do not
// displace one another in the caches, in a grid-stride loop over a fixed
// grid.  Elementwise arithmetic is fp32; the squared sums of one vector are
// added in fp32 and then into per-lane fp64 running sums.  The 2K+1 sums are
// reduced deterministically: halving exchanges in a wavefront, then the waves of the
// workgroup in order through LDS into one partial per workgroup (a plain
// store), then a second stage adds the partials in a fixed order: a one-workgroup
// kernel launched after this one on the same stream, or for the smallest calls the
// host, in that kernel's order.  With the grid fixed, every run adds the same
// numbers in the same order, so the statistics are bit-identical between runs.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "reduce.hpp"

namespace autoloco {

constexpr int kBlock = 256;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2r __attribute__((ext_vector_type(2)));

enum ReplicaType { RT_F32 = 0, RT_BF16 = 1 };
// Modes 5..8 are modes 1..4 with the worker average taken through BF16
// pseudo-gradient payloads.
enum Mode { MODE_STATS = 0, MODE_UPDATE = 1, MODE_UPDATE_STATS = 2, MODE_UPDATE_RESET = 3,
            MODE_UPDATE_STATS_RESET = 4, MODE_P_UPDATE = 5, MODE_P_UPDATE_STATS = 6, MODE_P_UPDATE_RESET = 7,
            MODE_P_UPDATE_STATS_RESET = 8, MODE_COUNT = 9 };

struct RoundArgs {
    float* theta;
    float* momentum;
    void* replicas[kMaxK];
    int64_t n;
    float mu, eta, scale, inv_k;
    double* partials;      // [2K+1][gridDim.x] per-workgroup sums
    uint16_t* payload;     // BF16 payload modes: [n] bits of the received mean, or null
    double inv_k64;        // 1/K in float64 (BF16 payload modes)
};

// ------------------------------------------------------------------ memory --
__device__ __forceinline__ f32x4 ld_f4(const float* p) {
    return __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
}
__device__ __forceinline__ void st_f4(float* p, f32x4 v) {
    __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(p));
}
__device__ __forceinline__ u32x4 ld_u4(const void* p) {
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}
__device__ __forceinline__ void st_u4(void* p, u32x4 v) {
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p));
}

// Same, at a wave-uniform base plus a 32-bit per-lane byte offset (lets the
// compiler keep the base in scalar registers).
__device__ __forceinline__ f32x4 ld_f4_at(const void* base, uint32_t off) {
    return __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(static_cast<const char*>(base) + off));
}
__device__ __forceinline__ void st_f4_at(void* base, uint32_t off, f32x4 v) {
    __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(static_cast<char*>(base) + off));
}
__device__ __forceinline__ u32x4 ld_u4_at(const void* base, uint32_t off) {
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(static_cast<const char*>(base) + off));
}
__device__ __forceinline__ void st_u4_at(void* base, uint32_t off, u32x4 v) {
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(static_cast<char*>(base) + off));
}
__device__ __forceinline__ u32x2r ld_u2_at(const void* base, uint32_t off) {
    return __builtin_nontemporal_load(reinterpret_cast<const u32x2r*>(static_cast<const char*>(base) + off));
}
__device__ __forceinline__ void st_u2_at(void* base, uint32_t off, u32x2r v) {
    __builtin_nontemporal_store(v, reinterpret_cast<u32x2r*>(static_cast<char*>(base) + off));
}

// bf16 <-> fp32.  Widening is exact.  Narrowing is gfx950's conversion
// instruction (one for a pair): round to nearest, ties to even, subnormals and
// infinities kept, overflow to infinity; a NaN stays a quiet NaN with the top
// of its payload.  (Over all 2^32 inputs other than NaN it gives the bits of
// the integer formulation (u + 0x7FFF + lsb) >> 16, checked on MI355X.)
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ uint32_t bf16_pack(float lo, float hi) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}
__device__ __forceinline__ uint32_t bf16_rne(float x) {
    return __builtin_bit_cast(uint16_t, static_cast<__bf16>(x));
}

// ------------------------------------------------------------- arithmetic --
template <int LO, int CNT, int K>
__device__ __forceinline__ float tree_sum(const float (&d)[K]) {
    if constexpr (CNT == 1) {
        return d[LO];
    } else {
        constexpr int H = CNT / 2;
        return tree_sum<LO, H, K>(d) + tree_sum<LO + H, CNT - H, K>(d);
    }
}

// One parameter: pseudo-gradients, their mean, the squared-sum terms and the
// corrected Nesterov step.  With BF16P the mean is the one every worker
// receives when the pseudo-gradients travel as BF16: each Delta_k rounded to
// BF16 (nearest even), their float64 sum in worker order times float64(1/K)
// rounded to FP32, then to BF16 (its bits go to pb); the squared sums use the
// unrounded Delta_k and that received mean.
// Only the fused multiply-adds written out are fused: without the pragma the
// compiler may fold the mean's product into Delta_k - mean in some kernel
// variants and not in others, and the standalone and fused statistics would
// then differ in their last bits.
template <int K, bool STATS, bool UPDATE, bool BF16P>
__device__ __forceinline__ void one_param(float th, float v, const float (&r)[K], const RoundArgs& a,
                                          float (&s)[K], float (&q)[K], float& m, float& th_new,
                                          float& v_new, uint32_t& pb) {
#pragma clang fp contract(off)
    float d[K];
#pragma unroll
    for (int k = 0; k < K; ++k) d[k] = th - r[k];
    float mean;
    if constexpr (BF16P) {
        double sum = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) sum += (double)__uint_as_float(bf16_rne(d[k]) << 16);
        pb = bf16_rne((float)(sum * a.inv_k64));
        mean = __uint_as_float(pb << 16);
    } else {
        mean = tree_sum<0, K, K>(d) * a.inv_k;
    }
    if constexpr (STATS) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            s[k] = __builtin_fmaf(d[k], d[k], s[k]);
            const float e = d[k] - mean;
            q[k] = __builtin_fmaf(e, e, q[k]);
        }
        m = __builtin_fmaf(mean, mean, m);
    }
    if constexpr (UPDATE) {
        const float dt = mean * a.scale;
        v_new = __builtin_fmaf(a.mu, v, dt);
        const float dir = __builtin_fmaf(a.mu, v_new, dt);
        th_new = __builtin_fmaf(-a.eta, dir, th);
    }
}

// Whole windows a workgroup keeps in flight (see the main loop).
//   Statistics only, which has no stores to overlap its loads with: about 256 bytes
//   of loads a lane, at most 8 windows.  384 to 768 bytes run alike at large sizes
//   and slower at small ones (10M, K = 8 bf16: 41 us at 256, 51 at 768).  Two windows
//   of 15 or 16 fp32 replicas, whose one is that much already: 300M, K = 15 2.87 ms
//   against 3.28 with one, 10M 106 us against 114.
//   The update with statistics and without the reset of up to 4 fp32 replicas, whose
//   one window a lane is too few loads for one workgroup a CU: about 160 bytes
//   (124M, K = 4: 0.79 ms with one window, 0.72 with two; 0.73 at three
//   workgroups a CU with one).
//   One otherwise: the reset's writes, or more replicas, keep the memory busy.
template <int K, int RT, bool STATS, bool UPDATE, bool RESET>
constexpr int windows_ahead() {
    const int bytes = RT == RT_F32 ? 16 * (K + 1) : 32 + 16 * K;
    if (!UPDATE && RT == RT_F32 && K >= 15) return 2;
    if (!UPDATE) return bytes >= 256 ? 1 : (256 + bytes - 1) / bytes > 8 ? 8 : (256 + bytes - 1) / bytes;
    if (RT == RT_F32 && STATS && !RESET && K <= 4) return (160 + 16 * (K + 2) - 1) / (16 * (K + 2));
    return 1;
}

// Workgroups up to which windows are kept in flight: one a compute unit for the update,
// three for the statistics alone.  Above (a caller's grid cap) there are waves enough,
// and with several windows each the memory runs worse: 124M fp32 at 1,024 workgroups,
// one window against several, statistics alone K = 1 145 us against 189, K = 8 0.64 ms
// against 0.80 (but K = 2 310 us against 276, and 251 against 293 at 2,048), the update
// with them K = 1 to 4 7-11 % faster.
constexpr unsigned ahead_grid(bool update) { return update ? 256 : 768; }

// ------------------------------------------------------------ round kernel --
template <int K, int RT, bool STATS, bool UPDATE, bool RESET, bool BF16P = false>
__global__ void __launch_bounds__(kBlock) round_kernel(RoundArgs a) {
    constexpr int NS = STATS ? 2 * K + 1 : 1;
    double acc[NS];
#pragma unroll
    for (int j = 0; j < NS; ++j) acc[j] = 0.0;

    // Parameters in runs of 4 ("quads": 16 bytes of fp32, 8 of bf16).  The
    // loop walks wave-uniform windows: each stream's window base stays in
    // scalar registers and a lane adds only its 32-bit offset.  fp32 replicas:
    // a lane owns one quad per window of 256; bf16 replicas: two, 256 quads
    // apart (a window of 512), so every load and store instruction of a
    // wavefront covers one contiguous run (1 KB of fp32, 512 B of bf16) and no
    // cache line is written in parts.
    constexpr int R = RT == RT_F32 ? 1 : 2;   // quads per lane per window
    constexpr int V = 4 * R;                  // parameters per lane per window
    const int64_t nq = a.n / 4;
    const int64_t qstride = (int64_t)gridDim.x * kBlock * R;
    const int64_t gtid = (int64_t)blockIdx.x * kBlock + threadIdx.x;

    // One window of a lane: its runs as loaded, and their arithmetic and stores.  ok1:
    // the second run of a bf16 window exists (in all but the last, shorter one).
    // bf16 replicas stay raw words until they are used, which leaves more loads in
    // flight (10M, K = 5, update with statistics: 49 us against 55); but widened run
    // by run in the update modes from K = 6 on, where at large sizes the memory runs
    // better with fewer (300M, K = 8: 1.63 ms against 1.77), and in the reset without
    // statistics, which gains nothing (1M, K = 4: 9.4 us against 10.6).
    constexpr bool RAW = RT == RT_BF16 && (!UPDATE || (K < 6 && (STATS || !RESET)));
    // The plain update of 12 or more fp32 replicas: all loads of a window ahead of the
    // first use, the momentum's last.  Left alone, the compiler moves loads behind the
    // first uses to save registers, and a window takes several trips to memory.
    // Kernel time: BF16 payload, 124M: K = 16 1.87 ms against 2.26, K = 15 1.73 against
    // 1.92; 10M, K = 14 126 us against 165.  Without it, 10M: K = 15 131 us against 141,
    // K = 14 125 against 148; K = 16 at 30M is 1 % slower.  Below 12 the compiler's order
    // is as fast or, at 124M and K = 9 to 11, 5 % faster.  The same for a single window of
    // the statistics alone of 15 or 16 (10,000 parameters, K = 15: 7.4 us against 8.2).
    constexpr bool TOGETHER = RT == RT_F32 && (UPDATE ? !STATS && !RESET && K >= 12 : K >= 15);
    // BF16 payload: the received mean goes out after theta and the momentum.  Stored
    // first, the wait for the last load of the window, the momentum's, was also a wait
    // for that store, and the window's other stores came only then.  (Fused with the
    // mean: fp32, 30M K = 2 171 us against 201, 124M K = 8 1.89 ms against 1.92; bf16, 30M
    // K = 7 248 us against 263.  Plain update of bf16 replicas: 124M K = 9 0.75 ms against
    // 0.80.)  First elsewhere, where the compiler then orders the loads better: 5 and 6
    // fp32 replicas fused run 1-3 % faster so at 30M to 124M, their update with statistics
    // or reset alone up to 10 %, and the rest alike.
    constexpr bool PAYLOAD_LAST = RT == RT_F32 ? STATS && RESET && K <= 8 && K != 5 && K != 6 : STATS == RESET && K >= 7;
    struct Window {
        f32x4 t[R], v[UPDATE ? R : 1];
        f32x4 rf[RAW ? 1 : K][RAW ? 1 : R];
        u32x2r rw[RAW ? K : 1][RAW ? R : 1];
    };
    auto load = [&](Window& w, int64_t qb, bool ok1) {
        const int64_t wb = qb * 4;                        // first parameter of the window
#pragma unroll
        for (int h = 0; h < R; ++h) {
            if (h == 1 && !ok1) {
                w.t[h] = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (UPDATE) w.v[h] = w.t[h];
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    if constexpr (RAW)
                        w.rw[k][h] = u32x2r{0u, 0u};
                    else
                        w.rf[k][h] = w.t[h];
                }
                continue;
            }
            const uint32_t fo = (h * kBlock + threadIdx.x) * 16u;   // byte offset in fp32 buffers
            w.t[h] = ld_f4_at(a.theta + wb, fo);
            if constexpr (UPDATE && !TOGETHER) w.v[h] = ld_f4_at(a.momentum + wb, fo);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if constexpr (RT == RT_F32) {
                    w.rf[k][h] = ld_f4_at(static_cast<const float*>(a.replicas[k]) + wb, fo);
                } else {
                    const u32x2r x = ld_u2_at(static_cast<const uint16_t*>(a.replicas[k]) + wb, fo / 2);
                    if constexpr (RAW)
                        w.rw[k][h] = x;
                    else
                        w.rf[k][h] = f32x4{bf16_lo(x[0]), bf16_hi(x[0]), bf16_lo(x[1]), bf16_hi(x[1])};
                }
            }
            if constexpr (TOGETHER) w.v[h] = ld_f4_at(a.momentum + wb, fo);
        }
    };
    auto step = [&](const Window& w, int64_t qb, bool ok1) {
        const int64_t wb = qb * 4;
        float* const th_w = a.theta + wb;
        float* const mo_w = a.momentum + wb;
        float s[K], q[K], m = 0.f;
#pragma unroll
        for (int k = 0; k < K; ++k) s[k] = q[k] = 0.f;
        float th_new[V], v_new[V];
        uint32_t pb[V];
#pragma unroll
        for (int e = 0; e < V; ++e) {
            float re[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if constexpr (!RAW)
                    re[k] = w.rf[k][e / 4][e & 3];
                else
                    re[k] = (e & 1) ? bf16_hi(w.rw[k][e / 4][(e & 3) >> 1]) : bf16_lo(w.rw[k][e / 4][(e & 3) >> 1]);
            }
            const float v = UPDATE ? w.v[UPDATE ? e / 4 : 0][e & 3] : 0.f;
            one_param<K, STATS, UPDATE, BF16P>(w.t[e / 4][e & 3], v, re, a, s, q, m, th_new[e], v_new[e], pb[e]);
        }
        if constexpr (STATS) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                acc[k] += (double)s[k];
                acc[K + k] += (double)q[k];
            }
            acc[2 * K] += (double)m;
        }
        if constexpr (!UPDATE) return;
#pragma unroll
        for (int h = 0; h < R; ++h) {
            if (h == 1 && !ok1) continue;
            const uint32_t fo = (h * kBlock + threadIdx.x) * 16u;
            auto store_payload = [&] {   // 2 bytes per parameter: 8 per quad
                if (a.payload != nullptr)
                    st_u2_at(a.payload + wb, fo / 2, u32x2r{pb[4 * h] | pb[4 * h + 1] << 16,
                                                            pb[4 * h + 2] | pb[4 * h + 3] << 16});
            };
            if constexpr (BF16P && !PAYLOAD_LAST) store_payload();
            const f32x4 o = {th_new[4 * h], th_new[4 * h + 1], th_new[4 * h + 2], th_new[4 * h + 3]};
            st_f4_at(th_w, fo, o);
            st_f4_at(mo_w, fo, f32x4{v_new[4 * h], v_new[4 * h + 1], v_new[4 * h + 2], v_new[4 * h + 3]});
            if constexpr (BF16P && PAYLOAD_LAST) store_payload();
            if constexpr (RESET) {
                if constexpr (RT == RT_F32) {
#pragma unroll
                    for (int k = 0; k < K; ++k) st_f4_at(static_cast<float*>(a.replicas[k]) + wb, fo, o);
                } else {
                    const u32x2r w2 = {bf16_pack(o[0], o[1]), bf16_pack(o[2], o[3])};
#pragma unroll
                    for (int k = 0; k < K; ++k) st_u2_at(static_cast<uint16_t*>(a.replicas[k]) + wb, fo / 2, w2);
                }
            }
        }
    };
    // Whole windows of the workgroup's grid-stride sequence, U of them in flight: each
    // is worked on in order (every sum as with one at a time) and the one U further
    // is loaded into its registers.
    constexpr int U = windows_ahead<K, RT, STATS, UPDATE, RESET>();
    int64_t qb = (int64_t)blockIdx.x * kBlock * R;
    if constexpr (U > 1) {
        if (gridDim.x <= ahead_grid(UPDATE) && qb + (U - 1) * qstride + kBlock * R <= nq) {
            Window w[U];
#pragma unroll
            for (int u = 0; u < U; ++u) load(w[u], qb + u * qstride, true);
            for (; qb + (2 * U - 1) * qstride + kBlock * R <= nq; qb += U * qstride) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    step(w[u], qb + u * qstride, true);
                    load(w[u], qb + (u + U) * qstride, true);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                step(w[u], qb + u * qstride, true);
                __builtin_amdgcn_sched_barrier(0);
            }
            qb += U * qstride;
        }
    }
    for (; qb < nq; qb += qstride) {
        if (qb + threadIdx.x >= nq) continue;
        const bool ok1 = R == 2 && qb + kBlock + threadIdx.x < nq;
        Window w;
        load(w, qb, ok1);
        if constexpr (TOGETHER) __builtin_amdgcn_sched_barrier(0);
        step(w, qb, ok1);
    }

    // Ragged tail: the last n mod 4 parameters, one per thread of workgroup 0.
    const int64_t tail0 = nq * 4;
    if (gtid < a.n - tail0) {
        const int64_t j = tail0 + gtid;
        const float th = a.theta[j];
        const float v = UPDATE ? a.momentum[j] : 0.f;
        float r[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if constexpr (RT == RT_F32)
                r[k] = static_cast<const float*>(a.replicas[k])[j];
            else
                r[k] = __uint_as_float((uint32_t) static_cast<const uint16_t*>(a.replicas[k])[j] << 16);
        }
        float s[K], q[K], m = 0.f, th_new = 0.f, v_new = 0.f;
        uint32_t pb = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) s[k] = q[k] = 0.f;
        one_param<K, STATS, UPDATE, BF16P>(th, v, r, a, s, q, m, th_new, v_new, pb);
        if constexpr (BF16P) {
            if (a.payload != nullptr) a.payload[j] = (uint16_t)pb;
        }
        if constexpr (STATS) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                acc[k] += (double)s[k];
                acc[K + k] += (double)q[k];
            }
            acc[2 * K] += (double)m;
        }
        if constexpr (UPDATE) {
            a.theta[j] = th_new;
            a.momentum[j] = v_new;
            if constexpr (RESET) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    if constexpr (RT == RT_F32)
                        static_cast<float*>(a.replicas[k])[j] = th_new;
                    else
                        static_cast<uint16_t*>(a.replicas[k])[j] = (uint16_t)bf16_rne(th_new);
                }
            }
        }
    }

    if constexpr (STATS) store_partials<NS, kBlock>(acc, a.partials);
}

// Launchers, one per (replica type, mode) translation unit.
typedef hipError_t (*RoundLauncher)(int k, int blocks, hipStream_t stream, const RoundArgs& a);
hipError_t launch_round_f32_m0(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_f32_m1(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_f32_m2(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_f32_m3(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_f32_m4(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_bf16_m0(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_bf16_m1(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_bf16_m2(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_bf16_m3(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_bf16_m4(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_f32_m5(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_f32_m6(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_f32_m7(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_f32_m8(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_bf16_m5(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_bf16_m6(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_bf16_m7(int, int, hipStream_t, const RoundArgs&);
hipError_t launch_round_bf16_m8(int, int, hipStream_t, const RoundArgs&);
// Resident workgroups per compute unit of the fused (update + stats + reset) kernel.
int occupancy_round_f32_m4(int k);
int occupancy_round_bf16_m4(int k);
int occupancy_round_f32_m8(int k);
int occupancy_round_bf16_m8(int k);

}  // namespace autoloco
