// Copying a table to LDS, for the kernels that probe staged tables.
#pragma once

#include "block.hpp"

namespace crystal {

// Copy a table of n words to LDS, 16 bytes per load and four loads per thread
// in flight (src is 16-byte aligned; dst, a multiple of 4 words).  Staging is a
// workgroup's start-up cost, bound by the latency of its loads: word by word it
// took 4 us more of a pass (16 star queries: 32.0 -> 28.8 us over 7.5M rows,
// 144.5 -> 139.9 us over 75M, with the first tile's load issued before it).
template <int BLOCK>
__device__ __forceinline__ void copy_to_lds(const uint32_t *__restrict__ src, uint32_t *__restrict__ dst, int n) {
    const v4i *s4 = reinterpret_cast<const v4i *>(src);
    v4i *d4 = reinterpret_cast<v4i *>(dst);
    const int n4 = n >> 2;
    int i = (int)threadIdx.x;
    for (; i + 3 * BLOCK < n4; i += 4 * BLOCK) {
        v4i x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = s4[i + k * BLOCK];
#pragma unroll
        for (int k = 0; k < 4; ++k) d4[i + k * BLOCK] = x[k];
    }
    for (; i < n4; i += BLOCK) d4[i] = s4[i];
    for (i = 4 * n4 + (int)threadIdx.x; i < n; i += BLOCK) dst[i] = src[i];
}

}  // namespace crystal
