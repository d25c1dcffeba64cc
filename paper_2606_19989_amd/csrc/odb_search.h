// The search of a run start in a rank's sorted lengths (odb_form.hip, chain_rank), apart from
// the kernels so that it can be checked on the host at sizes that no test window reaches.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace odb {

// Positions are unsigned: a rank holds up to 2^31 - 2 samples, so the sum of two positions, or a
// position rounded up to whole strides, may pass 2^31 but never 2^32.

// Distance of the sampled lengths: `samples` of them cover [0, last).
__host__ __device__ __forceinline__ uint32_t search_stride(uint32_t last, uint32_t samples) {
    return (last + samples - 1) / samples;
}

// First position p of [0, last) whose length is at most `at`, or `last`: len(p) does not increase
// with p, and sample(i) is len(i * stride), or 0 where that lies past the end.
template <typename Sample, typename Len>
__host__ __device__ __forceinline__ uint32_t first_at_most(const Sample& sample, const Len& len, uint32_t last,
                                                           uint32_t stride, uint32_t samples, int64_t at) {
    uint32_t lo = 0, hi = samples;   // first sample at or below the threshold
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (sample(mid) <= at) hi = mid; else lo = mid + 1;
    }
    // between sample lo - 1 (above) and sample lo
    uint32_t a = lo > 0 ? (lo - 1) * stride + 1 : 0;
    uint32_t z = lo * stride < last ? lo * stride : last;
    while (a < z) {
        const uint32_t mid = (a + z) >> 1;
        if (len(mid) <= at) z = mid; else a = mid + 1;
    }
    return a;
}

}  // namespace odb
