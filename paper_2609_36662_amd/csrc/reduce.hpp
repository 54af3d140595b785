// Deterministic reductions of per-thread fp64 sums, shared by the streaming
// kernels.  Every stage adds in a fixed order (halving exchanges inside a
// wavefront, the waves of a workgroup in index order through LDS, then the
// workgroups' partials in a fixed order in a one-workgroup finishing kernel, or for
// the smallest calls in that order on the host), so with a fixed grid the result is
// the same bit for bit on every run.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace autoloco {

constexpr int kMaxK = 16;
constexpr int kMaxSums = 2 * kMaxK + 1;

// One halving step on two sums: a lane whose bit of step S is clear returns a's
// value plus its partner's, the others b's.  Partners and bits: lane ^ 32 (bit 5),
// ^ 16 (4), ^ 8 (3), 7 - lane inside each 8 (bit 2), ^ 1 (0), ^ 2 (1).  The first
// two are gfx950's half and row swaps, which put both operands in place; the
// others choose what to send and exchange it with DPP.  Every lane must be active.
template <int S>
__device__ __forceinline__ double halve(double a, double b) {
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    if constexpr (S < 2) {
        auto swap = [](uint32_t p, uint32_t q) {
            if constexpr (S == 0)
                return __builtin_amdgcn_permlane32_swap(p, q, false, false);
            else
                return __builtin_amdgcn_permlane16_swap(p, q, false, false);
        };
        const auto lo = swap((uint32_t)x, (uint32_t)y), hi = swap((uint32_t)(x >> 32), (uint32_t)(y >> 32));
        return __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]) +
               __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
    } else {
        constexpr int bit = S == 2 ? 8 : S == 3 ? 4 : S == 4 ? 1 : 2;
        // row_ror:8, row_half_mirror, quad_perm 1,0,3,2, quad_perm 2,3,0,1
        constexpr int ctrl = S == 2 ? 0x128 : S == 3 ? 0x141 : S == 4 ? 0xB1 : 0x4E;
        const bool up = (threadIdx.x & bit) != 0;
        const uint64_t send = up ? x : y, keep = up ? y : x;
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)send, ctrl, 0xF, 0xF, false);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(send >> 32), ctrl, 0xF, 0xF, false);
        return __builtin_bit_cast(double, keep) + __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
    }
}

// The wavefront's total of sum wave_sum_of_lane(lane) (where that is below N): six
// halving steps, N - 1 + (odd counts) exchanges in all, where a butterfly per sum
// takes 6 N.
template <int N, int S = 0>
__device__ __forceinline__ double wave_sums(const double (&v)[N]) {
    if constexpr (S == 6) {
        static_assert(N == 1, "at most 64 sums");
        return v[0];
    } else {
        double w[(N + 1) / 2];
#pragma unroll
        for (int i = 0; i < N / 2; ++i) w[i] = halve<S>(v[2 * i], v[2 * i + 1]);
        if constexpr (N % 2 == 1) w[N / 2] = halve<S>(v[N - 1], v[N - 1]);
        return wave_sums<(N + 1) / 2, S + 1>(w);
    }
}
__device__ __forceinline__ int wave_sum_of_lane() {
    const int l = threadIdx.x & 63;
    return (l >> 5 & 1) + (l >> 4 & 1) * 2 + (l >> 3 & 1) * 4 + (l >> 2 & 1) * 8 + (l & 1) * 16 + (l >> 1 & 1) * 32;
}

// Sums acc[0..NS) over a workgroup of NT threads; thread j < NS returns sum j.
// Once per kernel (its LDS is not reused).
template <int NS, int NT>
__device__ __forceinline__ double block_reduce(const double (&acc)[NS]) {
    constexpr int NW = NT / 64;
    __shared__ double lds[NW * NS];
    const double v = wave_sums<NS>(acc);
    const int j = wave_sum_of_lane();
    if (j < NS) lds[(threadIdx.x >> 6) * NS + j] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x < NS) {
        t = lds[threadIdx.x];
#pragma unroll
        for (int w = 1; w < NW; ++w) t += lds[w * NS + threadIdx.x];
    }
    return t;
}

// Stage 1: this workgroup's sums into partials[NS][gridDim.x] (sum-major, so that
// stage 2 reads whole lines) with plain stores.  Stage 2 is finish_sums_kernel,
// launched after the producing kernel on the same stream (the stream order makes
// the partials visible to it), or the host once the stream has finished, where the
// partials are few and stored in its memory; so no workgroup takes a device-scope
// fence or a ticket at its end.  Latency-bound: a chain of exchanges, a round trip through
// LDS and one through memory.  A round of 10,000 parameters with statistics, both
// stages in it: K = 8 9.4 us, K = 16 11.1 (6.3 and 6.8 without statistics), against
// 13.4 and 18.8 with a butterfly per sum and workgroup-major partials.
template <int NS, int NT>
__device__ __forceinline__ void store_partials(const double (&acc)[NS], double* partials) {
    const double part = block_reduce<NS, NT>(acc);
    if (threadIdx.x < NS) partials[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = part;
}

// Stage 2, one workgroup of NT threads: thread t adds the partials of workgroups
// t, t + NT, ... in that order, then the workgroup reduces those as in stage 1;
// sums[0..NS) receives the totals.
template <int NS, int NT>
__global__ void __launch_bounds__(NT) finish_sums_kernel(const double* partials, int nblocks, double* sums,
                                                         double* host_copy) {
    double tot[NS];
#pragma unroll
    for (int j = 0; j < NS; ++j) tot[j] = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += NT) {
        double x[NS];
#pragma unroll
        for (int j = 0; j < NS; ++j) x[j] = partials[(int64_t)j * nblocks + b];
        __builtin_amdgcn_sched_barrier(0);   // all loads before the first add: one round trip, not NS
#pragma unroll
        for (int j = 0; j < NS; ++j) tot[j] += x[j];
    }
    const double fin = block_reduce<NS, NT>(tot);
    if (threadIdx.x < NS) {
        sums[threadIdx.x] = fin;
        if (host_copy != nullptr) host_copy[threadIdx.x] = fin;
    }
}

// Launches finish_sums_kernel for ns in 1..kMaxSums and nt in {256, 512};
// host_copy (may be null): a device view of coherent host memory that receives
// the sums as well, so no copy is needed to bring them to the host.
hipError_t launch_finish_sums(int ns, int nt, int nblocks, const double* partials, double* sums,
                              hipStream_t stream, double* host_copy = nullptr);

}  // namespace autoloco
