// Pieces of 16 bytes that were loaded so that they end where their row ends, put where they belong.
#pragma once
#include "gemm_kernel.h"

namespace fact {

// 8 elements shifted down by s elements (element e <- element e + s), zeros from the top; s >= 8 gives zeros
__device__ __forceinline__ u32x4_t shift_down(u32x4_t v, int s)
{
    const int w = s >> 1;
    u32x4_t r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t x = 0;
#pragma unroll
        for (int j = i; j < 4; ++j) x = w == j - i ? v[j] : x;
        r[i] = x;
    }
    if (s & 1) {
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = (r[i] >> 16) | (i < 3 ? r[i < 3 ? i + 1 : 3] << 16 : 0u);
    }
    return r;
}

}  // namespace fact
