// For tests/test_gpu_head_widths.py: the bf16 parts of floats as the score and matching kernels split them.
#include "../paper_2406_18139_amd/csrc/frag.h"

// x: groups of eight floats; dots, differences, half: twelve words a group, three parts of four pairs each
__global__ void __launch_bounds__(256) k_split(const float* __restrict__ x, int groups, uint32_t* dots, uint32_t* differences, uint32_t* half)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= groups) return;
    const lookm::frag_f32 lo = reinterpret_cast<const lookm::frag_f32*>(x)[2 * i], hi = reinterpret_cast<const lookm::frag_f32*>(x)[2 * i + 1];
    const lookm::frag_split s[3] = {lookm::split_steps<true, true>(lo, hi), lookm::split_steps<true, false>(lo, hi), lookm::split_steps<false, true>(lo, hi)};
    uint32_t* out[3] = {dots, differences, half};
    for (int n = 0; n < 3; ++n)
        for (int part = 0; part < 3; ++part) reinterpret_cast<lookm::frag_words*>(out[n])[3 * i + part] = s[n].w[part];
}

extern "C" int split_check(const float* x, int groups, uint32_t* dots, uint32_t* differences, uint32_t* half, void* stream)
{
    if (!x || !dots || !differences || !half || groups <= 0) return -1;
    hipLaunchKernelGGL(k_split, dim3((groups + 255) / 256), dim3(256), 0, (hipStream_t)stream, x, groups, dots, differences, half);
    return hipPeekAtLastError() == hipSuccess ? 0 : -6;
}
