// Bit-matrix helpers shared by kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace homs {

// transposes a 32 x 32 bit matrix held as 32 words: bit i of word j becomes
// bit j of word i (swaps of bit blocks of 16, 8, 4, 2, 1)
__device__ __forceinline__ void transpose32(uint32_t (&v)[32])
{
    uint32_t mask = 0x0000FFFFu;
#pragma unroll
    for (int j = 16; j > 0; j >>= 1) {
#pragma unroll
        for (int k = 0; k < 32; ++k)
            if ((k & j) == 0) {
                const uint32_t t = ((v[k] >> j) ^ v[k + j]) & mask;
                v[k + j] ^= t;
                v[k] ^= t << j;
            }
        mask ^= mask << (j >> 1);
    }
}

}  // namespace homs
