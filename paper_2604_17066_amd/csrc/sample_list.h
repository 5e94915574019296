// The list of unclassified samples: k_label appends the indices that a block
// finds to a region of that block and leaves the region's extent, so that the
// list needs no counter (one to clear before, and atomics on one address) and is in
// sample order.  A reader forms the prefix sums of the extents first.
#pragma once

#include "rsr_internal.h"

namespace rsr {

// before[r] = listed samples in the regions before r, before[kListRegions] =
// all of them.  Every thread of the block must call it; the first wave works.
__device__ __forceinline__ uint32_t list_prefix(const SampleList& list, uint32_t* before) {
    constexpr int kPer = kListRegions / 64;
    if (threadIdx.x < 64) {
        uint32_t n[kPer], sum = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            n[k] = static_cast<uint32_t>(list.regions[threadIdx.x * kPer + k].y);
            sum += n[k];
        }
        uint32_t run = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t o = __shfl_up(run, d);
            if (static_cast<int>(threadIdx.x) >= d) run += o;
        }
        if (threadIdx.x == 63) before[kListRegions] = run;
        run -= sum;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            before[threadIdx.x * kPer + k] = run;
            run += n[k];
        }
    }
    __syncthreads();
    return before[kListRegions];
}

// Entry j < total of the list.
__device__ __forceinline__ int64_t list_at(const SampleList& list, const uint32_t* before,
                                           uint32_t j) {
    int a = 0, b = kListRegions - 1;
    while (a < b) {
        const int m = (a + b + 1) >> 1;
        if (before[m] <= j) a = m;
        else b = m - 1;
    }
    return list.index[static_cast<int64_t>(list.regions[a].x) + (j - before[a])];
}

}  // namespace rsr
