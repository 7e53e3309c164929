// What the kernels over 4 x 4 groups of C blocks share: the work item of a
// workgroup, reductions over a wave, and launches of any number of groups.
#pragma once

#include <algorithm>

#include "smm.h"

namespace bsm {

// Work item of this workgroup, -1 for none: the launch's items (a.q_count
// groups from a.q_first on, as far as there are groups) form kXcds contiguous
// ranges, one per XCD (as in the quad kernel).
__device__ inline int64_t group_item(const SmmArgs &a) {
    const int64_t left = (a.n_quads_dev ? *a.n_quads_dev : a.n_quads) - a.q_first;
    const int64_t n = left < a.q_count ? left : a.q_count;
    const int64_t per = (n + kXcds - 1) / kXcds;
    if (static_cast<int64_t>(blockIdx.x / kXcds) >= per) return -1;
    const int64_t it = static_cast<int64_t>(blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
    return it < n ? a.q_first + it : -1;
}

__device__ inline double group_wave_sum(double v) {
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}
__device__ inline double group_wave_max(double v) {
    for (int o = kWave / 2; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, kWave));
    return v;
}

// launch(args, grid) over all groups, one workgroup of `threads` each, in
// slices of fewer than 2^32 threads (the most that one launch may have).
template <class F>
int launch_groups(const SmmArgs &a, int threads, F launch) {
    const int64_t most = ((int64_t{1} << 32) / threads - 1) / kXcds * kXcds;
    for (int64_t first = 0; first < a.n_quads; first += most) {
        SmmArgs b = a;
        b.q_first = first;
        b.q_count = std::min(most, a.n_quads - first);
        launch(b, static_cast<unsigned>((b.q_count + kXcds - 1) / kXcds * kXcds));
        BSM_HIP(hipGetLastError());
    }
    return BSM_OK;
}

}  // namespace bsm
