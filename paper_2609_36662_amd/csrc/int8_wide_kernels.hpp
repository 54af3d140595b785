// The INT8-codec round (see int8_kernels.hpp for its arithmetic) for 9 to 16
// workers, on gfx950.
//
// One workgroup of 512 threads owns one codec block of 4,096 parameters at a
// time, 8 parameters a thread.  The K pseudo-gradients of a block are used
// three times with a workgroup barrier between the uses (local energy and block
// maxima; codes; deviations from the aggregate), so they have to stay on the
// chip: K * 16 KB, 256 KB at K = 16.  They live in registers, K * 8 of the 256 a
// thread of an 8-wave workgroup may use, and everything else is arranged
// around that:
//   - the next block comes in while this one is encoded: theta and the replicas
//     by direct global-to-LDS loads (all of bf16, the first 8 of fp32: 144 KB of
//     the CU's 160), workers 9 and up of fp32 into the registers that the
//     deviations have just freed;
//   - a thread keeps one fp64 accumulator for four sums (quad_add);
//   - theta leaves the registers while the codes are formed and is read from its
//     LDS piece again for the update.
// Bound by HBM traffic as the round is.  GPT-2 small, K = 16 fp32, encoded mean
// written (18.0 GB): 3.30 ms, 5.5 TB/s, against 8.2-8.9 ms for the kernel for up
// to 8 workers, whose registers spill here (1.1 KB of scratch a thread) and which
// has no prefetch above 8 workers.
#pragma once

#include "int8_kernels.hpp"

namespace autoloco {

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

template <int K, int RT, bool STATS, bool RESET>
__global__ void __launch_bounds__(kInt8Threads) int8_wide_kernel(Int8Args a) {
    static_assert(K > 8 && K <= 16, "9 to 16 workers");
    constexpr int NT = kInt8Threads;
    constexpr int NW = NT / 64;
    constexpr int V = 8, G = 2, W = V / G;       // two runs of 4 parameters a thread, 2,048 apart
    constexpr int NS = 2 * K + 1;
    constexpr int Q4 = (K + 3) / 4;              // groups of four workers
    // workers whose next block streams into LDS; the rest of fp32 replicas (8
    // bytes a thread and run more than 160 KB hold) come through registers
    constexpr int LK = RT == RT_F32 ? 8 : K;
    constexpr int RK = K - LK;
    constexpr int RV = RT == RT_F32 ? G * NT : NT;   // 16-byte vectors of one replica's block
    __shared__ uint32_t lds_max[2 * 8 * kWorkerMaxStride(NW)];
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
    auto to_lds = [&](const void* base, uint32_t off, int vec) {
        __builtin_amdgcn_global_load_lds(
            (const void __attribute__((address_space(1)))*)(static_cast<const char*>(base) + off),
            (void __attribute__((address_space(3)))*)(lds_pf + vec + wave * 64), 16, 0, 0);
    };
    // Issues the direct loads of full block b: theta's, and the replicas'.
    auto pf_theta = [&](int64_t b) {
#pragma unroll
        for (int g = 0; g < G; ++g) to_lds(fbase(a.theta, b, g), fo, g * NT);
    };
    auto pf_replicas = [&](int64_t b) {
        if constexpr (RT == RT_F32) {
            uint32_t o = fo;
            asm volatile("" : "+v"(o));   // no per-lane sums kept across the loop
#pragma unroll
            for (int k = 0; k < LK; ++k)
#pragma unroll
                for (int g = 0; g < G; ++g) to_lds(fbase(a.replicas[k], b, g), o, G * NT + k * RV + g * NT);
        } else {
            // lanes 0..31 the wave's first run (512 B), lanes 32..63 its second
            uint32_t ro = (lane >> 5) * kCodecBlock + wave * 512u + (lane & 31) * 16u;
            asm volatile("" : "+v"(ro));
#pragma unroll
            for (int k = 0; k < LK; ++k) to_lds(bbase(a.replicas[k], b, 0), ro, G * NT + k * RV);
        }
    };
    f32x4 nx[RK > 0 ? RK : 1][G];   // the next block's vectors of workers LK..K-1
    auto reg_issue = [&](int64_t b, int k) {
#pragma unroll
        for (int g = 0; g < G; ++g) nx[k - LK][g] = ld_f4_at(fbase(a.replicas[k], b, g), fo);
    };

    auto body = [&](int64_t blk, auto full_c) {
        constexpr bool FULL = decltype(full_c)::value;
        const int64_t nb = blk + gridDim.x < nfull ? blk + gridDim.x : blk;
        int64_t off[G];
        int valid[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            off[g] = blk * kCodecBlock + g * (kCodecBlock / 2) + (int64_t)threadIdx.x * W;
            const int64_t left = a.n - off[g];
            valid[g] = FULL || left >= W ? W : (left > 0 ? (int)left : 0);
        }
        float th[V], v[V], d[K][V];
        if constexpr (FULL) {
            // This block's direct loads were issued in the previous iteration (or
            // before the loop), and the last vector memory instructions issued
            // after them are that iteration's stores: G of theta, G of v and, with
            // the reset, G of each replica.  In-order completion makes "at most
            // that many outstanding" imply the loads have landed in LDS.
            constexpr int after = G * (2 + (RESET ? K : 0));
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(after) : "memory");
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
            // direct loads overwrite the pieces (on the workgroup's last block this
            // block again, so that every iteration issues the same instructions;
            // those values are not used)
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            pf_replicas(nb);
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

        // worker block maxima: lane l gets worker (l mod 16)'s
        float amax[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            float m = 0.f;
            if (k < K) {
#pragma unroll
                for (int e = 0; e < V; ++e) m = fmaxf(m, fabsf(d[k][e]));
            }
            amax[k] = m;
        }
        const float am = worker_block_max16<NW>(amax, lds_max);
        // momentum: in flight while the codes are formed
        if constexpr (FULL) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const f32x4 v4 = ld_f4_at(fbase(a.momentum, blk, g), fo);
#pragma unroll
                for (int e = 0; e < W; ++e) v[g * W + e] = v4[e];
            }
        }
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
        float mmax[1] = {0.f};
#pragma unroll
        for (int e = 0; e < V; ++e) {
            mean[e] = (float)(sum[e] * a.inv_k);
            mmax[0] = fmaxf(mmax[0], fabsf(mean[e]));
        }
        block_max<1, NT, true>(mmax, lds_mmax);
        const float sm = codec_scale(mmax[0]);
        const float rm = 1.0f / sm;

        float agg[V], qm[V];
        codec_q<V>([&](int e) { return mean[e]; }, sm, rm, qm);
#pragma unroll
        for (int e = 0; e < V; ++e) agg[e] = FULL || e % W < valid[e / W] ? qm[e] * sm : 0.0f;

        if constexpr (FULL) {
            // theta is read from LDS again (its registers served the codes meanwhile);
            // its next block may then be loaded there.  The momentum is waited for
            // before any further load is issued.
            uint32_t li = threadIdx.x;
            asm volatile("" : "+v"(li));
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const f32x4 t4 = lds_pf[g * NT + li];
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    th[g * W + e] = t4[e];
                    asm volatile("" : "+v"(v[g * W + e]));
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            pf_theta(nb);
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
                    if (4 * j + i >= LK && 4 * j + i < K) reg_issue(nb, 4 * j + i);
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
        pf_theta(blockIdx.x);
        pf_replicas(blockIdx.x);
#pragma unroll
        for (int k = LK; k < K; ++k) reg_issue(blockIdx.x, k);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the first block's pieces are in LDS
    for (int64_t blk = blockIdx.x; blk < nfull; blk += gridDim.x) body(blk, BoolC<true>{});
    // the last iteration's direct loads (a re-read, unused) land before anything
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

}  // namespace autoloco
