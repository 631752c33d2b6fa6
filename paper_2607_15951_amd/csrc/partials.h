// partials.h -- the view counters from the projection's per-block sums: by a
// kernel of their own (project.hip), or by the first workgroups of the depth
// sort's first launch, which saves a launch and its wait.
#pragma once

#include "gs_internal.h"

namespace gsmi {

// The counters of view v, summed over the projection blocks' partials by the
// kThreads threads of a workgroup.  With changed, also the items whose key or
// rectangle changed (added over the views; each view's share clamped to
// 2^32 - 1), clearing the flag that none did when any did.
template <int kThreads>
__device__ __forceinline__ void sum_partials(const PartialSums& a, int v)
{
    // 64-bit sums: in each thread over a stride of blocks, in each wave by
    // shuffles, then over the waves in LDS
    constexpr int kWaves = kThreads / 64;
    __shared__ unsigned long long s_sum[kWaves][6];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long t[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll 4
    for (int b = threadIdx.x; b < a.blocks; b += kThreads) {
        const uint4* pp = reinterpret_cast<const uint4*>(a.partials + kPartials * ((int64_t)b * a.n_views + v));
        const uint4 lo = pp[0];
        const uint2 hi = *reinterpret_cast<const uint2*>(pp + 1);
        t[0] += lo.x;
        t[1] += lo.y;
        t[2] += lo.z;
        t[3] += lo.w;
        t[4] += hi.x;
        t[5] += hi.y;
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        for (int o = 32; o > 0; o >>= 1) t[k] += __shfl_xor(t[k], o, 64);
        if (lane == 0) s_sum[wave][k] = t[k];
    }
    __syncthreads();
    if (threadIdx.x < kViewCounters) {   // one thread per counter
        // its sum, and whether the counter is that sum's upper half
        const int k = threadIdx.x, of = k == 0 ? 0 : (k == 1 ? 2 : (k < 4 ? 1 : (k < 6 ? 4 : (k < 8 ? 5 : 3))));
        unsigned long long sum = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) sum += s_sum[w][of];
        uint32_t c = (k == 3 || k == 5 || k == 7) ? (uint32_t)(sum >> 32) : (uint32_t)sum;
        const uint32_t moved = !a.changed || k != 8 ? 0u : (sum > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)sum);
        if (k >= 8) c = moved;   // the last counter is spare
        a.view_counts[(int64_t)kViewCounters * v + k] = c;
        // may be pinned host memory, read after an event past the kernel
        if (a.counts_out) a.counts_out[(int64_t)kViewCounters * v + k] = c;
        if (moved) {
            // views add their counts; any change clears the flag (all
            // writers store the same 0)
            atomicAdd(&a.changed[0], moved);
            a.changed[1] = 0u;
        }
    }
}

}  // namespace gsmi
