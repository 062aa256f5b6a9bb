// What the score passes of score_mfma.hip leave behind for the kernels after them.
#pragma once
#include "common.h"

namespace lookm {

constexpr int SD = 128;        // head dim
constexpr int BS = 256;        // stationary rows per workgroup
constexpr int BX = 64;         // streamed rows per iteration
constexpr int LIST_HEAD = 64;  // lists[0], lists[1]: number of competing and of protected keys; the lists themselves from here on

// First chunk of `CT` streamed rows that a strip of competing keys has partials of; p_strip: the strip's first position.
__device__ __forceinline__ int sparse_first_chunk(int p_strip, int R0, int CT) { return max((p_strip / BX) * BX, (R0 / BX) * BX) / CT; }

// Inverse norms of the protected keys of head h, which pass 2 over the competing keys does not hold: eight lanes per key, lane p
// summing the dims 8p .. 8p+7 and 64+8p .. 64+8p+7 in order, then a pairwise tree - the order of the stand-alone norm kernel, so
// that both give the same bits.  Group `first` of eight threads takes the keys first, first + step, ...
__device__ __forceinline__ void protected_norms(const int32_t* __restrict__ lists, int h, int L, const bf16_t* __restrict__ k,
                                                float* __restrict__ rnorm, int first, int step)
{
    const int NP = lists[1], sub = threadIdx.x & 7;
    for (int idx = first; idx < NP; idx += step) {     // uniform per group of eight lanes
        const int pos = lists[LIST_HEAD + L + idx];
        const bf16_t* row = k + ((size_t)h * L + pos) * SD;
        double ss = 0.0;
#pragma unroll
        for (int rep = 0; rep < 2; ++rep) {
            float v[8];
            load8(row + sub * 8 + rep * 64, v);
#pragma unroll
            for (int i = 0; i < 8; ++i) ss = fma((double)v[i], (double)v[i], ss);
        }
        ss += __shfl_xor(ss, 1);
        ss += __shfl_xor(ss, 2);
        ss += __shfl_xor(ss, 4);
        if (sub == 0) rnorm[(size_t)h * L + pos] = inverse_norm(ss);
    }
}

}  // namespace lookm
