// A synchronisation round whose pseudo-gradient average travels through the
// INT8 blockwise codec (App. G.1), on gfx950.
//
// One workgroup of 512 threads owns one codec block of 4,096 parameters at a
// time (8 parameters per thread), so every buffer is still read once and
// written once.  Per block:
//   Delta_k = theta - theta_k                                (fp32)
//   S_k += Delta_k^2                 D is measured before quantisation
//   s_k = max|Delta_k| / 127 (1 for a zero block, at least 2^-126)
//   q = clip(rne(Delta_k / s_k), -127, 127);  Delta^_k = q s_k    (fp32)
//   mean = fp32(sum_k Delta^_k (fp64, worker order) * fp64(1/K))
//   the mean is encoded and decoded once more (same rule)  -> Delta_agg
//   Q_k += (Delta_k - Delta_agg)^2, M += Delta_agg^2          C uses the aggregate
//   corrected Nesterov step with Delta_agg, reset of the replicas
// The two block maxima (the K worker maxima, then the mean's) are exact and
// order-independent: lane exchanges (DPP) inside each wavefront, then the
// waves through LDS, with one barrier each.
// Every codec step runs in fp32 with IEEE division and round-to-nearest-even,
// so the codes are the same integers the FP32 definition gives.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "reduce.hpp"
#include "round_kernels.hpp"

namespace autoloco {

constexpr int kCodecBlock = 4096;

struct Int8Args {
    float* theta;
    float* momentum;
    void* replicas[kMaxK];
    int64_t n;
    float mu, eta, scale;
    double inv_k;
    int8_t* mean_codes;   // [n] or null
    float* mean_scales;   // [ceil(n / 4096)] or null
    double* partials;     // [2K+1][gridDim.x] per-workgroup sums
};

__device__ __forceinline__ float codec_scale(float amax) {
    if (amax == 0.0f) return 1.0f;
    const float s = amax / 127.0f;
    return s < 0x1p-126f ? 0x1p-126f : s;
}

// Codes of x[0..NV) at scale s (r = fp32(1/s)): the integers nearest
// fp32(x / s), ties to even, clipped to +-127.  t = x * r differs from
// fp32(x / s) by at most (3u + u^2) |x / s| <= 2.28e-5 here (u = 2^-24,
// |x / s| <= 127.00003), so rint(t) is the same integer unless t lies within
// 3e-5 of a half-integer; only then (about 6e-5 of the elements) is the IEEE
// quotient formed.  t - rint(t) is exact (Sterbenz); where the compiler fuses
// the product into it, the test value is x r - rint(t) rounded once, within
// u |x / s| of the exact one, which the margin covers as well.  The common path
// has no per-element test: each lane keeps the largest |t - rint(t)| of its
// elements, and one wavefront-uniform branch leads to the quotients when some
// lane's exceeds the bound.  A NaN t drops out of that maximum, which is
// harmless: t is NaN only when x is NaN, or infinite in a block whose scale is
// infinite (r = 0), and the quotient is NaN then too.
// The clip is implied by the scale and costs no instruction: s is the block's
// largest magnitude over 127 rounded once (or the larger 2^-126), so |t| and
// |fp32(x / s)| are at most 127 (1 + 3 * 2^-24) < 127.5 for every x of the
// block, and their nearest integers lie in [-127, 127].  (A non-finite block
// has an infinite scale and decodes to non-finite values either way.)
// x(e) gives element e (evaluated again on the rare path).
template <int NV, typename X>
__device__ __forceinline__ void codec_q(X x, float s, float r, float (&q)[NV]) {
    constexpr float kNear = 0.5f - 3.0e-5f;
    float dev = 0.0f;
#pragma unroll
    for (int e = 0; e < NV; ++e) {
        const float t = x(e) * r;
        q[e] = __builtin_rintf(t);
        dev = fmaxf(dev, fabsf(t - q[e]));
    }
    if (__builtin_amdgcn_ballot_w64(dev >= kNear) != 0) {
#pragma unroll
        for (int e = 0; e < NV; ++e)
            if (!(fabsf(x(e) * r - q[e]) < kNear)) q[e] = __builtin_rintf(x(e) / s);
    }
}

// Maximum over the 64 lanes of a wavefront of a non-negative float (or NaN),
// compared as its bit pattern, which orders non-negative floats as numbers:
// DPP exchanges within each row of 16 lanes, then the four row results are read
// out as wave-uniform values.
__device__ __forceinline__ uint32_t wave_max_bits(uint32_t x) {
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, false));   // quad_perm 2,3,0,1
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, false));  // row_half_mirror
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xF, 0xF, false));  // row_mirror
    const uint32_t a = max((uint32_t)__builtin_amdgcn_readlane((int)x, 0), (uint32_t)__builtin_amdgcn_readlane((int)x, 16));
    const uint32_t b = max((uint32_t)__builtin_amdgcn_readlane((int)x, 32), (uint32_t)__builtin_amdgcn_readlane((int)x, 48));
    return max(a, b);
}

// Workgroup barrier that waits for this wave's LDS traffic only.  __syncthreads
// would also wait for every direct global-to-LDS load in flight, which the
// prefetch of the next block is.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Maximum of a non-negative value over the workgroup (every thread gets it).
// One barrier: the caller gives each use within a loop iteration its own LDS
// region, so a wave that runs ahead into the next iteration writes a region
// every other wave has finished reading (they all passed a later barrier of
// this iteration after reading it).  Every thread of the workgroup must be
// active.
template <int NT>
__device__ __forceinline__ void block_max(float& v, uint32_t* lds) {
    constexpr int NW = NT / 64;
    const uint32_t m = wave_max_bits(__float_as_uint(v));
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = m;
    lds_barrier();
    uint32_t x = lds[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) x = max(x, lds[w]);
    v = __uint_as_float(x);
}

// Block maxima of up to 16 workers' non-negative values (compared as their bit
// patterns) over a workgroup of NW waves, in groups of 8 workers; returns
// worker (lane mod 8)'s in every lane, or above 8 workers (lane mod 16)'s.
// Instead of one wavefront reduction per worker, a halving exchange inside each
// group of 8 lanes (partners 7 - i, i ^ 1, i ^ 2; every lane sends the half of
// its values its partner keeps) leaves lane i with the group's maximum of worker
// w(i) = 4 b2 + 2 b0 + b1 (b_j the bits of i), a rotation by 8 lanes joins the
// two groups of each row of 16, and every wave stores its 4 row values per
// worker.  After the one barrier each lane reads the 4 NW values of its worker
// (rows 16-byte aligned, 4 words apart in bank order, so the 8 workers' reads
// fall in distinct banks).  The same reuse rule as block_max holds for the LDS
// region.
constexpr int kWorkerMaxStride(int nw) { return 4 * nw + 4; }

// Stores this wave's 4 row maxima of each of 8 workers.
template <int NW>
__device__ __forceinline__ void worker_max_rows(const uint32_t (&m)[8], uint32_t* lds) {
    constexpr int S = kWorkerMaxStride(NW);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool lo = (lane & 4) == 0, even = (lane & 1) == 0, b1 = (lane & 2) != 0;
    uint32_t a4[4], a2[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {   // partner 7 - i (row_half_mirror): the low lane keeps workers 0..3
        const uint32_t send = lo ? m[j + 4] : m[j], keep = lo ? m[j] : m[j + 4];
        a4[j] = max(keep, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)send, 0x141, 0xF, 0xF, false));
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {   // partner i ^ 1 (quad_perm 1,0,3,2)
        const uint32_t send = even ? a4[j + 2] : a4[j], keep = even ? a4[j] : a4[j + 2];
        a2[j] = max(keep, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)send, 0xB1, 0xF, 0xF, false));
    }
    uint32_t c;
    {                               // partner i ^ 2 (quad_perm 2,3,0,1)
        const uint32_t send = b1 ? a2[0] : a2[1], keep = b1 ? a2[1] : a2[0];
        c = max(keep, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)send, 0x4E, 0xF, 0xF, false));
    }
    c = max(c, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0x128, 0xF, 0xF, false));   // row_ror:8
    const int w = (lane & 4) + ((lane & 1) << 1) + ((lane & 2) >> 1);
    if ((lane & 8) == 0) lds[w * S + wave * 4 + (lane >> 4)] = c;
}

template <int K, int NW>
__device__ __forceinline__ float worker_block_max(const float (&v)[K], uint32_t* lds) {
    static_assert(K <= 16, "at most 16 workers");
    constexpr int S = kWorkerMaxStride(NW), H = K <= 8 ? 1 : 2;
#pragma unroll
    for (int h = 0; h < H; ++h) {
        uint32_t m[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) m[j] = 8 * h + j < K ? __float_as_uint(v[8 * h + j < K ? 8 * h + j : 0]) : 0u;
        worker_max_rows<NW>(m, lds + h * 8 * S);
    }
    lds_barrier();
    const uint32_t* p = lds + (threadIdx.x & (8 * H - 1)) * S;
    uint32_t r = 0;
#pragma unroll
    for (int i = 0; i < 4 * NW; ++i) r = max(r, p[i]);
    return __uint_as_float(r);
}

constexpr int kInt8Threads = 512;  // one codec block of 4,096 parameters per workgroup

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <bool B>
struct BoolC {
    static constexpr bool value = B;
};

// Adds x[0..3] to four fp64 sums over all lanes, in one fp64 accumulator a lane:
// lane i keeps sum i mod 4, adding the four values of its quad (two exchanges:
// partners i ^ 1, then i ^ 2).
__device__ __forceinline__ void quad_add(double& acc, float x0, float x1, float x2, float x3) {
    const bool odd = (threadIdx.x & 1) != 0, hi = (threadIdx.x & 2) != 0;
    auto pair = [&](float a, float b) {
        const float send = odd ? a : b, keep = odd ? b : a;
        return (double)keep + (double)__int_as_float(__builtin_amdgcn_update_dpp(
                                  0, __float_as_int(send), 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
    };
    const double p = pair(x0, x1), q = pair(x2, x3);
    const uint64_t send = __builtin_bit_cast(uint64_t, hi ? p : q);
    const uint32_t lo32 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)send, 0x4E, 0xF, 0xF, false);
    const uint32_t hi32 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(send >> 32), 0x4E, 0xF, 0xF, false);
    acc += (hi ? q : p) + __builtin_bit_cast(double, (uint64_t)hi32 << 32 | lo32);   // quad_perm 2,3,0,1
}

// Each thread of a workgroup owns 8 parameters of a codec block: two runs of
// 4, 2,048 apart, so every wavefront instruction covers one contiguous run
// (1 KB of fp32, 512 B of bf16) and no cache line is written in parts.  The loop
// runs over the full blocks, in which every load and store is a whole vector;
// the one shorter last block, if any, goes through a second instance of the same
// body with per-element accesses.
//
// The K pseudo-gradients of a block are used three times with a workgroup barrier
// between the uses (local energy and block maxima; codes; deviations from the
// aggregate), so they have to stay on the chip: K * 16 KB, 256 KB at K = 16.  They
// live in registers, K * 8 of the 256 a thread of an 8-wave workgroup may use, and
// the rest is arranged around that:
//   - the next block comes in while this one is encoded, theta and the replicas
//     by direct global-to-LDS loads (no registers; each wave into pieces only it
//     reads back, behind an explicit count of the vector memory instructions
//     issued after them, since the compiler does not order these loads against
//     later LDS reads by itself), fp32 workers 9 and up into the registers that
//     the deviations have just freed;
//   - the block barriers wait for LDS traffic only, not for those loads;
//   - a thread keeps one fp64 accumulator for four sums (quad_add);
//   - above 8 workers theta leaves the registers while the codes are formed and is
//     read from its LDS piece again for the update.
// Bound by HBM traffic as the round is, at one workgroup a CU.  Kernel time, plain
// torch allocations, caches flushed, against the kernel before it (the next block
// of bf16 replicas in registers and fp64 sums in LDS; fp32's in LDS, but waited
// for at the first barrier and without the non-temporal hint; no prefetch and
// 1.1 KB of scratch a thread at K = 16):
//   GPT-2 small, K = 16 fp32, encoded mean (18.0 GB): 3.3-3.6 ms from 8.2-8.9 ms
//   100M, K = 8 fp32 (8.0 GB): 1.55 ms from 1.67; without the reset 0.81 from 0.91
//   100M, K = 8 bf16 (4.8 GB): 0.93 ms alike; without the reset 0.575 from 0.625
//   8M, K = 8 fp32 / bf16: 146 / 95 us from 171 / 104
template <int K, int RT, bool STATS, bool RESET>
__global__ void __launch_bounds__(kInt8Threads) int8_round_kernel(Int8Args a) {
    constexpr int NT = kInt8Threads;
    constexpr int NW = NT / 64;
    constexpr int V = 8, G = 2, W = V / G;       // two runs of 4 parameters a thread, 2,048 apart
    constexpr int NS = 2 * K + 1;
    constexpr int Q4 = (K + 3) / 4;              // groups of four workers
    // workers whose next block streams into LDS (with theta up to 144 KB of the
    // CU's 160); fp32 workers 9 and up come through registers
    constexpr int LK = RT == RT_F32 && K > 8 ? 8 : K;
    constexpr int RK = K - LK;
    constexpr int RV = RT == RT_F32 ? G * NT : NT;   // 16-byte vectors of one replica's block
    // theta stays in registers over the codes up to 8 workers; above, it is read
    // from its LDS piece again for the update
    constexpr bool KEEP_THETA = K <= 8;
    // The momentum's loads go out while the codes are formed; with the reset and 4
    // to 8 bf16 workers, before the next block's (100M, K = 8: 0.928 ms against
    // 0.975, K = 4: 0.574 against 0.600; without the reset 0.603 against 0.575, and
    // fp32 replicas run alike either way).
    constexpr bool EARLY_V = RESET && RT == RT_BF16 && K >= 4 && K <= 8;
    __shared__ uint32_t lds_max[(K <= 8 ? 8 : 16) * kWorkerMaxStride(NW)];
    __shared__ uint32_t lds_mmax[NW];
    // [theta: run][wave][lane], then [replica][run][wave][lane] (bf16: a wave's
    // two 512-byte runs in one 1 KB piece); every wave reads back only the 1 KB
    // pieces it loaded itself
    __shared__ f32x4 lds_pf[G * NT + LK * RV];

    double acc_s[STATS ? Q4 : 1], acc_q[STATS ? Q4 : 1], acc_m = 0.0;
#pragma unroll
    for (int j = 0; j < (STATS ? Q4 : 1); ++j) acc_s[j] = acc_q[j] = 0.0;

    const int64_t nfull = a.n / kCodecBlock;
    const int64_t nblocks = (a.n + kCodecBlock - 1) / kCodecBlock;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;

    // Streams are addressed as a wave-uniform base (block and run) plus a 32-bit
    // lane offset, and the LDS pieces as one lane index plus constants: neither
    // leaves a per-lane pointer for each stream alive across the loop.
    const uint32_t fo = threadIdx.x * 16u;        // byte offset of a thread's run in fp32 streams
    auto fbase = [](const void* p, int64_t blk, int g) {
        return static_cast<const char*>(p) + (blk * kCodecBlock + g * (kCodecBlock / 2)) * 4;
    };
    auto bbase = [](const void* p, int64_t blk, int g) {
        return static_cast<const char*>(p) + (blk * kCodecBlock + g * (kCodecBlock / 2)) * 2;
    };
    // non-temporal (the last operand's bit 1), as every other access of the round: 5-30 % of the
    // whole call on streams that no cache holds (8M, K = 8 fp32, no reset: 90 us
    // against 130), and never slower than before where one does
    auto to_lds = [&](const void* base, uint32_t off, int vec) {
        __builtin_amdgcn_global_load_lds(
            (const void __attribute__((address_space(1)))*)(static_cast<const char*>(base) + off),
            (void __attribute__((address_space(3)))*)(lds_pf + vec + wave * 64), 16, 0, 2);
    };
    // Issues the direct loads of full block b: theta's, and the replicas'.
    auto pf_theta = [&](int64_t b, uint32_t lanes) {
#pragma unroll
        for (int g = 0; g < G; ++g) to_lds(fbase(a.theta, b, g), fo & lanes, g * NT);
    };
    auto pf_replicas = [&](int64_t b, uint32_t lanes) {
        if constexpr (RT == RT_F32) {
            uint32_t o = fo & lanes;
            asm volatile("" : "+v"(o));   // no per-lane sums kept across the loop
#pragma unroll
            for (int k = 0; k < LK; ++k)
#pragma unroll
                for (int g = 0; g < G; ++g) to_lds(fbase(a.replicas[k], b, g), o, G * NT + k * RV + g * NT);
        } else {
            // lanes 0..31 the wave's first run (512 B), lanes 32..63 its second
            uint32_t ro = ((lane >> 5) * kCodecBlock + wave * 512u + (lane & 31) * 16u) & lanes;
            asm volatile("" : "+v"(ro));
#pragma unroll
            for (int k = 0; k < LK; ++k) to_lds(bbase(a.replicas[k], b, 0), ro, G * NT + k * RV);
        }
    };
    f32x4 nx[RK > 0 ? RK : 1][G];   // the next block's vectors of workers LK..K-1
    auto reg_issue = [&](int64_t b, uint32_t lanes, int k) {
#pragma unroll
        for (int g = 0; g < G; ++g) nx[k - LK][g] = ld_f4_at(fbase(a.replicas[k], b, g), fo & lanes);
    };

    auto body = [&](int64_t blk, auto full_c) {
        constexpr bool FULL = decltype(full_c)::value;
        // The workgroup's next block.  On its last one the loads are issued all the same
        // (a branch around them takes up to 30 registers more, and K = 15 and 16 spill),
        // but all lanes of a load then read the same 16 bytes, the first of this block's
        // run, and nothing uses them: this block read once more cost a sixth of the call
        // where a workgroup has one block (1M, K = 12 fp32 with the reset and without
        // statistics: 28 us against 33; 4M 97 against 104).
        const bool more = blk + gridDim.x < nfull;
        const int64_t nb = more ? blk + gridDim.x : blk;
        const uint32_t lanes = more ? ~0u : 0u;
        int64_t off[G];
        int valid[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            off[g] = blk * kCodecBlock + g * (kCodecBlock / 2) + (int64_t)threadIdx.x * W;
            const int64_t left = a.n - off[g];
            valid[g] = FULL || left >= W ? W : (left > 0 ? (int)left : 0);
        }
        float th[V], v[V], d[K][V];
        // momentum, first needed by the update
        auto load_v = [&] {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const f32x4 v4 = ld_f4_at(fbase(a.momentum, blk, g), fo);
#pragma unroll
                for (int e = 0; e < W; ++e) v[g * W + e] = v4[e];
            }
        };
        if constexpr (FULL) {
            // This block's direct loads were issued in the previous iteration (or
            // before the loop), and the last vector memory instructions issued
            // after them are that iteration's stores: G of theta, G of v and, with
            // the reset, G of each replica.  In-order completion makes "at most
            // that many outstanding" imply the loads have landed in LDS.
            constexpr int after = G * (2 + (RESET ? K : 0));
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(after) : "memory");
            if constexpr (EARLY_V) load_v();
            uint32_t li = threadIdx.x;
            asm volatile("" : "+v"(li));
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const f32x4 t4 = lds_pf[g * NT + li];
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    th[g * W + e] = t4[e];
                }
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    if constexpr (RT == RT_F32) {
                        const f32x4 r4 = k < LK ? lds_pf[G * NT + k * RV + g * NT + li] : nx[k < LK ? 0 : k - LK][g];
#pragma unroll
                        for (int e = 0; e < W; ++e) d[k][g * W + e] = th[g * W + e] - r4[e];
                    } else {
                        const u32x2 w = reinterpret_cast<const u32x2*>(lds_pf + G * NT + k * RV)[g * 64 + (li >> 6) * 128 + (li & 63)];
#pragma unroll
                        for (int e = 0; e < W; ++e)
                            d[k][g * W + e] = th[g * W + e] - ((e & 1) ? bf16_hi(w[e >> 1]) : bf16_lo(w[e >> 1]));
                    }
                }
            }
            // every LDS read of this block has returned before the next block's
            // direct loads overwrite the pieces
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if constexpr (KEEP_THETA) pf_theta(nb, lanes);
            pf_replicas(nb, lanes);
        } else {
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    const bool in = e < valid[g];
                    const int x = g * W + e;
                    const int64_t o = off[g] + e;
                    th[x] = in ? a.theta[o] : 0.0f;
                    v[x] = in ? a.momentum[o] : 0.0f;
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        float r = 0.0f;
                        if (in) {
                            if constexpr (RT == RT_F32)
                                r = static_cast<const float*>(a.replicas[k])[o];
                            else
                                r = __uint_as_float((uint32_t) static_cast<const uint16_t*>(a.replicas[k])[o] << 16);
                        }
                        d[k][x] = th[x] - r;
                    }
                }
        }

        // local-drift energy before quantisation
        if constexpr (STATS) {
#pragma unroll
            for (int j = 0; j < Q4; ++j) {
                float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (4 * j + i < K) {
#pragma unroll
                        for (int e = 0; e < V; ++e) s[i] = __builtin_fmaf(d[4 * j + i][e], d[4 * j + i][e], s[i]);
                    }
                quad_add(acc_s[j], s[0], s[1], s[2], s[3]);
            }
        }

        // worker block maxima: lane l gets worker (l mod 8)'s, or above 8 workers (l mod 16)'s
        float amax[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            float m = 0.f;
#pragma unroll
            for (int e = 0; e < V; ++e) m = fmaxf(m, fabsf(d[k][e]));
            amax[k] = m;
        }
        const float am = worker_block_max<K, NW>(amax, lds_max);
        if constexpr (FULL && !EARLY_V) load_v();
        // one division of each kind for all workers: lane k computes worker k's
        const float sv = codec_scale(am);
        const float rv = 1.0f / sv;

        // decode every worker and average: fp64 sum in worker order, times fp64(1/K)
        double sum[V];
#pragma unroll
        for (int e = 0; e < V; ++e) sum[e] = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const float s = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sv), k));
            const float r = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(rv), k));
            float q[V];
            codec_q<V>([&](int e) { return d[k][e]; }, s, r, q);
#pragma unroll
            for (int e = 0; e < V; ++e) {
                sum[e] += (double)(q[e] * s);
                // the sum is taken here: left alone, the compiler moves every worker's
                // additions past the codec's branches to one place at the end and keeps
                // all K * 8 codes in registers until then
                asm volatile("" : "+v"(sum[e]));
            }
        }
        float mean[V];
        float mmax = 0.f;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            mean[e] = (float)(sum[e] * a.inv_k);
            mmax = fmaxf(mmax, fabsf(mean[e]));
        }
        block_max<NT>(mmax, lds_mmax);
        const float sm = codec_scale(mmax);
        const float rm = 1.0f / sm;

        float agg[V], qm[V];
        codec_q<V>([&](int e) { return mean[e]; }, sm, rm, qm);
#pragma unroll
        for (int e = 0; e < V; ++e) agg[e] = FULL || e % W < valid[e / W] ? qm[e] * sm : 0.0f;

        if constexpr (FULL) {
            // the momentum is waited for before any further load is issued
#pragma unroll
            for (int e = 0; e < V; ++e) asm volatile("" : "+v"(v[e]));
        }
        if constexpr (FULL && !KEEP_THETA) {
            uint32_t li = threadIdx.x;
            asm volatile("" : "+v"(li));
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const f32x4 t4 = lds_pf[g * NT + li];
#pragma unroll
                for (int e = 0; e < W; ++e) th[g * W + e] = t4[e];
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            pf_theta(nb, lanes);
        }

        // deviations from the aggregate; a worker's pseudo-gradients are not used
        // after this, so its next block can be loaded into their registers
#pragma unroll
        for (int j = 0; j < Q4; ++j) {
            if constexpr (STATS) {
                float q[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (4 * j + i < K) {
#pragma unroll
                        for (int e = 0; e < V; ++e) {
                            const float t = d[4 * j + i][e] - agg[e];
                            q[i] = __builtin_fmaf(t, t, q[i]);
                        }
                    }
                quad_add(acc_q[j], q[0], q[1], q[2], q[3]);
            }
            if constexpr (FULL && RK > 0) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (4 * j + i >= LK && 4 * j + i < K) reg_issue(nb, lanes, 4 * j + i);
            }
        }
        if constexpr (STATS) {
            float m = 0.f;
#pragma unroll
            for (int e = 0; e < V; ++e) m = __builtin_fmaf(agg[e], agg[e], m);
            acc_m += (double)m;
        }

        if (a.mean_codes != nullptr) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (FULL || valid[g] == W) {
                    uint32_t w = 0;
#pragma unroll
                    for (int e = 0; e < W; ++e) w |= (uint32_t)(uint8_t)(int8_t)qm[g * W + e] << (8 * e);
                    __builtin_nontemporal_store(w, reinterpret_cast<uint32_t*>(a.mean_codes + off[g]));
                } else {
#pragma unroll
                    for (int e = 0; e < W; ++e)
                        if (e < valid[g]) a.mean_codes[off[g] + e] = (int8_t)qm[g * W + e];
                }
            }
            if (threadIdx.x == 0) a.mean_scales[blk] = sm;
        }

        // corrected Nesterov step with the decoded aggregate, and the reset
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int64_t o = off[g];
            float tn[W], vn[W];
#pragma unroll
            for (int e = 0; e < W; ++e) {
                const int x = g * W + e;
                const float dt = agg[x] * a.scale;
                vn[e] = __builtin_fmaf(a.mu, v[x], dt);
                const float dir = __builtin_fmaf(a.mu, vn[e], dt);
                tn[e] = __builtin_fmaf(-a.eta, dir, th[x]);
            }
            if (FULL || valid[g] == W) {
                const f32x4 t4 = {tn[0], tn[1], tn[2], tn[3]};
                st_f4_at(const_cast<char*>(fbase(a.theta, blk, g)), fo, t4);
                st_f4_at(const_cast<char*>(fbase(a.momentum, blk, g)), fo, f32x4{vn[0], vn[1], vn[2], vn[3]});
                if constexpr (RESET) {
                    if constexpr (RT == RT_F32) {
#pragma unroll
                        for (int k = 0; k < K; ++k) st_f4_at(const_cast<char*>(fbase(a.replicas[k], blk, g)), fo, t4);
                    } else {
                        const u32x2 w = {bf16_pack(tn[0], tn[1]), bf16_pack(tn[2], tn[3])};
#pragma unroll
                        for (int k = 0; k < K; ++k)
                            st_u2_at(const_cast<char*>(bbase(a.replicas[k], blk, g)), fo / 2, w);
                    }
                }
            } else {
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    if (e < valid[g]) {
                        a.theta[o + e] = tn[e];
                        a.momentum[o + e] = vn[e];
                        if constexpr (RESET) {
#pragma unroll
                            for (int k = 0; k < K; ++k) {
                                if constexpr (RT == RT_F32)
                                    static_cast<float*>(a.replicas[k])[o + e] = tn[e];
                                else
                                    static_cast<uint16_t*>(a.replicas[k])[o + e] = (uint16_t)bf16_rne(tn[e]);
                            }
                        }
                    }
                }
            }
        }
    };

    if (blockIdx.x < nfull) {
        pf_theta(blockIdx.x, ~0u);
        pf_replicas(blockIdx.x, ~0u);
#pragma unroll
        for (int k = LK; k < K; ++k) reg_issue(blockIdx.x, ~0u, k);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the first block's pieces are in LDS
    for (int64_t blk = blockIdx.x; blk < nfull; blk += gridDim.x) body(blk, BoolC<true>{});
    // the last iteration's direct loads (unused) land before anything
    // else uses this workgroup's LDS or the workgroup ends
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // the shorter last block belongs to the workgroup the grid stride gives it
    if (nfull < nblocks && nfull % gridDim.x == blockIdx.x) body(nfull, BoolC<false>{});

    if constexpr (STATS) {
        // back to one value per sum and lane (a sum's other lanes hold zeros)
        const int mine = threadIdx.x & 3;
        double r[NS];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            r[k] = mine == k % 4 ? acc_s[k / 4] : 0.0;
            r[K + k] = mine == k % 4 ? acc_q[k / 4] : 0.0;
        }
        r[2 * K] = acc_m;
        store_partials<NS, NT>(r, a.partials);
    }
}

typedef hipError_t (*Int8Launcher)(int k, int blocks, hipStream_t stream, const Int8Args& a);
// one per (replica type, stats, reset): launch_int8_<rt>_s<stats>r<reset>
hipError_t launch_int8_f32_s0r0(int, int, hipStream_t, const Int8Args&);
hipError_t launch_int8_f32_s0r1(int, int, hipStream_t, const Int8Args&);
hipError_t launch_int8_f32_s1r0(int, int, hipStream_t, const Int8Args&);
hipError_t launch_int8_f32_s1r1(int, int, hipStream_t, const Int8Args&);
hipError_t launch_int8_bf16_s0r0(int, int, hipStream_t, const Int8Args&);
hipError_t launch_int8_bf16_s0r1(int, int, hipStream_t, const Int8Args&);
hipError_t launch_int8_bf16_s1r0(int, int, hipStream_t, const Int8Args&);
hipError_t launch_int8_bf16_s1r1(int, int, hipStream_t, const Int8Args&);

}  // namespace autoloco
