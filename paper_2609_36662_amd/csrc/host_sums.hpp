// The second stage of the reductions on the host (plain C++, no device code), for
// calls whose per-workgroup sums are few enough that adding them here is cheaper
// than a second launch.
#pragma once

#include <cstdint>

namespace autoloco {

// Stage 2 of the reduction on the host, in finish_sums_kernel's order (thread t of nt
// adds the workgroups t, t + nt, ...; then the exchanges of wave_sums, lane distances
// 32, 16, 8, the half-row mirror, 1 and 2; then the wavefronts in order), so the sums
// have that kernel's bits: partials[ns][nblocks] into sums[0..ns).
inline void host_finish_sums(const double* partials, int ns, int nt, int nblocks, double* sums) {
    for (int j = 0; j < ns; ++j) {
        const double* p = partials + static_cast<int64_t>(j) * nblocks;
        double total = 0.0;
        for (int w = 0; w * 64 < nt && (w == 0 || w * 64 < nblocks); ++w) {
            double x[64] = {};
            for (int b = w * 64; b < nblocks; b += nt)
                for (int i = 0; i < 64 && b + i < nblocks; ++i) x[i] += p[b + i];
            for (int d = 32; d >= 8; d /= 2)
                for (int i = 0; i < d; ++i) x[i] += x[i + d];
            for (int i = 0; i < 4; ++i) x[i] += x[7 - i];
            const double wave = (x[0] + x[1]) + (x[2] + x[3]);
            total = w == 0 ? wave : total + wave;
        }
        sums[j] = total;
    }
}

}  // namespace autoloco
