// Operand fragments of the 16x16 matrix instructions for any head width (the score and matching kernels in
// score_any.hip / nearest_any.hip).
//
// One step of a fragment is 16 bytes per lane: lane (c = lane % 16, q = lane / 16) holds, of row c, eight
// consecutive bf16 (dims 32*ks + 8q, one v_mfma_f32_16x16x32_bf16) or four consecutive floats (dims 16*ks + 4q, four
// v_mfma_f32_16x16x4_f32, number i taking element i of every lane: the dims are visited in another order than they are
// stored in, the same one for both operands).  Products of bf16 pairs are exact and fp32 ones are fused
// multiply-adds; both accumulate in fp32.
//
// All rows pass through LDS on their way to registers: lanes of equal q hold
// different rows, so a fragment read from global memory touches 16 cache lines for 1 KB and runs at a quarter of the
// L1 rate (measured: scores of 32 heads x 2781 x 64 bf16, 44 us a pass; with 32 stationary rows per wave instead of
// 64, i.e. twice the loads, 66 us).  A wave copies its block of 32 rows with coalesced direct-to-LDS loads into a
// buffer of its own - no barrier - and reads the fragments from there; the buffer is free again as soon as they are
// in registers, so one buffer per wave is enough to have the next block in flight.
#pragma once
#include "common.h"

#include <type_traits>

namespace lookm {

typedef __attribute__((ext_vector_type(8))) __bf16 frag_bf16;
typedef __attribute__((ext_vector_type(4))) float frag_f32;
typedef __attribute__((ext_vector_type(4))) float acc_t;

template <typename T> struct frag;
template <> struct frag<bf16_t> {
    typedef frag_bf16 type;
    static constexpr int WIDTH = 8;     // dims per lane and step
    static constexpr int SUB = 1;       // matrix instructions per step
    static __device__ __forceinline__ acc_t mma(int, type a, type b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};
template <> struct frag<float> {
    typedef frag_f32 type;
    static constexpr int WIDTH = 4;
    static constexpr int SUB = 4;
    static __device__ __forceinline__ acc_t mma(int i, type a, type b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], c, 0, 0, 0);
    }
};

// Row of an LDS block: KS steps of 64 bytes, rounded up to a power of two.
template <int KS> constexpr int frag_row_bytes() { return KS <= 1 ? 64 : KS <= 2 ? 128 : KS <= 4 ? 256 : KS <= 8 ? 512 : 1024; }
constexpr int FRAG_BLOCK = 32;     // rows

// Where chunk `chunk` (16 bytes) of row r sits in its LDS row: sixteen-byte reads of eight consecutive rows at the same
// chunk hit all banks once.
template <int KS>
__device__ __forceinline__ int frag_swizzle(int chunk, int r)
{
    return frag_row_bytes<KS>() >= 128 ? chunk ^ (r & 7) : chunk ^ ((r >> 1) & 3);
}

// Copies ROWS rows to LDS: 1 KB per instruction, lane l of instruction n filling the 16 bytes number 64n + l.
// row_of(r) gives the byte offset of the block's row r from `base` (below 2^32).  The chunks of a padded row that lie
// past the end of the head width repeat its first one; frag_read puts zeros there.
template <typename T, int KS, int ROWS, typename RowOf>
__device__ __forceinline__ void frag_load_block(const T* __restrict__ base, int d, void* lds, int lane, RowOf&& row_of)
{
    constexpr int RB = frag_row_bytes<KS>(), CH = RB / 16, NI = ROWS * RB / 1024;
    const char* b = reinterpret_cast<const char*>(base);
    const int chunks = d * (int)sizeof(T) / 16;
#pragma unroll
    for (int n = 0; n < NI; ++n) {
        const int s = n * 64 + lane, r = s / CH;
        int c = frag_swizzle<KS>(s % CH, r);       // the swizzle is its own inverse
        c = (c < chunks) ? c : 0;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(b + (row_of(n, r) + (uint32_t)(c * 16))),
                                         (__attribute__((address_space(3))) void*)((char*)lds + n * 1024), 16, 0, 0);
    }
}
// The same for consecutive rows of a tensor, through a buffer descriptor: what a lane adds to the scalar offset of the first row
// depends on the piece only through its place in the swizzle's pattern of eight rows, so that loading a block takes no address
// arithmetic (row_of takes six instructions a piece, which for 32 x 2781 x 64 bf16 was a sixth of a score pass's vector
// instructions).
template <int KS> constexpr int frag_row_kinds() { return frag_row_bytes<KS>() <= 128 ? 1 : frag_row_bytes<KS>() / 128; }
template <typename T, int KS>
__device__ __forceinline__ void frag_row_offsets(int d, int lane, int* off)
{
    constexpr int CH = frag_row_bytes<KS>() / 16;
    const int chunks = d * (int)sizeof(T) / 16;
#pragma unroll
    for (int v = 0; v < frag_row_kinds<KS>(); ++v) {
        const int r = v * (64 / CH) + lane / CH, c = frag_swizzle<KS>(lane % CH, r);
        off[v] = r * d * (int)sizeof(T) + (c < chunks ? c * 16 : 0);
    }
}
// ROWS rows from row0 on, the first `rows` of them inside the tensor (scalar values); the others repeat its last row
template <typename T, int KS, int ROWS>
__device__ __forceinline__ void frag_load_rows(__amdgpu_buffer_rsrc_t rsrc, int d, void* lds, int lane, const int* off,
                                               int row0, int rows)
{
    constexpr int RB = frag_row_bytes<KS>(), CH = RB / 16, NI = ROWS * RB / 1024, V = frag_row_kinds<KS>();
    static_assert(NI >= 1, "");
    const int row_bytes = d * (int)sizeof(T);
    if (rows >= ROWS) {
#pragma unroll
        for (int n = 0; n < NI; ++n)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)((char*)lds + n * 1024), 16, off[n % V],
                                                     (row0 + n / V * V * (64 / CH)) * row_bytes, 0, 0);
    } else {
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int r = n * (64 / CH) + lane / CH, past = min(rows - 1 - r, 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)((char*)lds + n * 1024), 16,
                                                     off[n % V] + (row0 + n / V * V * (64 / CH) + past) * row_bytes, 0, 0, 0);
        }
    }
}
// The fragments of rows 16*rg + c of a block.  Past the head width they are zeros like the stationary operand's: what the
// block repeats there may hold an infinity, and 0 * inf would turn a logit of -inf into NaN.
template <typename T, int KS>
__device__ __forceinline__ void frag_read(const void* lds, int rg, int c16, int q4, int d, typename frag<T>::type (&a)[KS])
{
    const char* row = (const char*)lds + (16 * rg + c16) * frag_row_bytes<KS>();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        a[ks] = *reinterpret_cast<const typename frag<T>::type*>(row + frag_swizzle<KS>(ks * 4 + q4, c16) * 16);
    if (d < KS * 4 * frag<T>::WIDTH) {             // uniform: widths that fill their steps pay a scalar branch
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            if ((ks * 4 + q4) * frag<T>::WIDTH >= d) a[ks] = typename frag<T>::type{};
    }
}
// Rows of a strip of 16 * CG stationary rows that a wave loads: a quarter, but 1 KB at least and whole patterns of the swizzle.
template <int KS, int CG> constexpr int frag_strip_part() { return (frag_row_bytes<KS>() == 64 || CG == 4) ? 16 : 8; }
// Everything a wave has asked for has arrived: direct-to-LDS loads are not tracked by the compiler.
__device__ __forceinline__ void frag_wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }     // vmcnt(0)

// inverse norms of the rows 32*block .. 32*block + 31 of k ([rows, d]) by a workgroup of 256 threads: eight lanes per
// row, lane p summing the dims 8p .. 8p+7, 64+8p .., in order, then a pairwise tree.  The squares are summed in
// binary64 (for bf16 keys every square and, in practice, every partial sum is exact), so that the result is the
// correctly rounded inverse norm up to one final rounding: the matching on the matrix cores budgets half a unit in
// the last place for this factor.
template <typename T>
__device__ __forceinline__ void inverse_norms(const T* __restrict__ k, size_t rows, int d, size_t block, float* __restrict__ rnorm)
{
    const size_t row = block * 32 + (threadIdx.x >> 3);
    const int sub = threadIdx.x & 7;
    double s = 0.0;
    if (row < rows) {
        for (int c0 = sub * 8; c0 < d; c0 += 64) {
            float v[8];
            load8(k + row * d + c0, v);
            for (int i = 0; i < 8; ++i) s = fma((double)v[i], (double)v[i], s);
        }
    }
    s += __shfl_xor(s, 1);
    s += __shfl_xor(s, 2);
    s += __shfl_xor(s, 4);
    if (row < rows && sub == 0) rnorm[row] = inverse_norm(s);
}

// Calls f(steps, groups) with integral constants: the steps of a fragment that hold d dims, and how many groups of 16
// stationary rows a wave keeps in registers next to them: as many as 64 registers hold (at most 4 groups, 2 for fp32,
// whose matrix instructions take eight times as long per LDS byte) - or a single group where such strips would leave
// most of the chip idle: strips(rows per strip), fewer than one per compute unit.  The score passes count the strips of
// the query heads for both: with grouped heads pass 2 has fewer workgroups than that, each with several heads to go
// through (32 query heads on 8 key heads x 700 x 64 bf16: 88 for 256 compute units; not tuned).  (A 256-token fp32 prompt of 2 x 64: score passes and matching 21 us with two groups, 16 us with one; 1483 tokens of 16 x 128, 750
// workgroups: 163 us with two groups, 168 us with one, and a tenth of the LDS traffic more per flop than that shows.)
template <typename T, typename Strips, typename F>
inline void with_frag_shape(int d, Strips&& strips, F&& f)
{
    constexpr int per_step = 4 * frag<T>::WIDTH, cg_max = (sizeof(T) == 2) ? 4 : 2;
    const int ks = (d + per_step - 1) / per_step;
    auto go = [&](auto steps) {
        constexpr int KS = decltype(steps)::value, CG = (4 * KS * cg_max <= 64) ? cg_max : cg_max / 2;
        if (CG > 1 && strips(16 * CG) < 256) f(steps, std::integral_constant<int, 1>{});
        else f(steps, std::integral_constant<int, CG>{});
    };
    if (ks <= 1) go(std::integral_constant<int, 1>{});
    else if (ks <= 2) go(std::integral_constant<int, 2>{});
    else if (ks <= 3) go(std::integral_constant<int, 3>{});
    else if (ks <= 4) go(std::integral_constant<int, 4>{});
    else if (ks <= 6) go(std::integral_constant<int, 6>{});
    else if (ks <= 8) go(std::integral_constant<int, 8>{});
    else if constexpr (sizeof(T) == 4) {
        if (ks <= 12) go(std::integral_constant<int, 12>{});
        else go(std::integral_constant<int, 16>{});
    }
}

}  // namespace lookm
