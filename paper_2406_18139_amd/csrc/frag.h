// Operand fragments of the 16x16 matrix instructions for any head width (the score and matching kernels in
// score_any.hip / nearest_any.hip).
//
// One step of a fragment is 16 bytes per lane: lane (c = lane % 16, q = lane / 16) holds, of row c, eight
// consecutive bf16 (dims 32*ks + 8q, one v_mfma_f32_16x16x32_bf16) or four consecutive floats (dims 16*ks + 4q; the dims
// are multiplied in another order than they are stored in, the same one for both operands).  Products of bf16 pairs are
// exact; everything accumulates in fp32.  For fp32 see frag_split.
//
// All rows pass through LDS on their way to registers: lanes of equal q hold different rows, so a fragment read from
// global memory touches 16 cache lines for 1 KB and runs at a quarter of the L1 rate (measured: scores of 32 heads x 2781 x 64 bf16, 44 us a pass; with 32 stationary rows per wave instead of
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
};
template <> struct frag<float> {
    typedef frag_f32 type;
    static constexpr int WIDTH = 4;
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
        // The row number is hidden from the compiler: where a piece is a row (fp32 wider than 128) it would otherwise carry one
        // counter per piece through the caller's loop, 32 of them and more than the scalar registers hold (16 x 1483 x 136:
        // pass 2 119 us, 108 without them; in narrower ones vector registers, 10 to 60 of them).
        int last = rows - 1;
        asm volatile("" : "+s"(last));
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int r = n * (64 / CH) + lane / CH, past = min(last - r, 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)((char*)lds + n * 1024), 16,
                                                     off[n % V] + (row0 + n / V * V * (64 / CH) + past) * row_bytes, 0, 0, 0);
        }
    }
}
// The fragments of rows 16*rg + c of a block.  Past the head width they are zeros like the stationary operand's: what the
// block repeats there may hold an infinity, and 0 * inf would turn a logit of -inf into NaN.  Only the steps past the next
// smaller fragment can hold such dims.  The words are selected whole: selected as eight bf16 the compiler takes them
// apart and puts them together again, two instructions a word in every block (32 x 2781 x 72: 143 us the whole layer, 121 with
// whole words).
template <int KS> constexpr int frag_full_steps() { return KS <= 4 ? KS - 1 : KS <= 8 ? KS - 2 : KS - 4; }     // see with_frag_shape
template <typename T, int KS>
__device__ __forceinline__ void frag_read(const void* lds, int rg, int c16, int q4, int d, typename frag<T>::type (&a)[KS])
{
    const char* row = (const char*)lds + (16 * rg + c16) * frag_row_bytes<KS>();
    typedef __attribute__((ext_vector_type(4))) uint32_t words;
    words w[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) w[ks] = *reinterpret_cast<const words*>(row + frag_swizzle<KS>(ks * 4 + q4, c16) * 16);
    if (d < KS * 4 * frag<T>::WIDTH) {             // uniform: widths that fill their steps pay a scalar branch
#pragma unroll
        for (int ks = frag_full_steps<KS>(); ks < KS; ++ks)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if ((ks * 4 + q4) * frag<T>::WIDTH >= d) w[ks][i] = 0;
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) a[ks] = __builtin_bit_cast(typename frag<T>::type, w[ks]);
}
// fp32 products on the bf16 matrix instruction, which is sixteen times as fast as the fp32 one.  A float is the sum of three
// bf16 values, each the remainder's nearest: 24 bits exactly.  Of the nine products of two such sums the six largest are
// added up, smallest first, and the sum is rounded in fp32 once per 32 dims of every kind where the fp32 instruction rounds once
// per 4 dims.  What is left out is just over 2^-26 of the product at most, with either sign, and nothing of a product that fits into 24
// bits (both factors need more than 8, one more than 16).  Against binary64, 32 heads x 700 and 12 to 60 seeds of each width and
// distribution, parts / fp32 instruction: scores rms 1.68e-7 / 1.68e-7 (8 dims), 1.70e-7 / 1.73e-7 (64), 1.70e-7 / 1.75e-7 (128), of sharp
// softmax rows 1.9e-7 / 2.2e-7, 3.2e-7 / 6.1e-7, 3.6e-7 / 8.1e-7; the largest of a seed, on average, 8.1e-7 / 8.3e-7, 7.8e-7 / 9.4e-7,
// 7.7e-7 / 1.07e-6; cosines rms 4.8e-8 / 5.6e-8, 2.3e-8 / 4.6e-8, 1.9e-8 / 4.4e-8.  (All nine products: the same to three digits, and 15 %
// of the time of a 1483 x 128 layer more.)  Two steps of four floats make one step of eight bf16 dims.
//
// What the parts cannot hold goes to the fp32 instruction.  An infinity in a streamed row, or a value that rounds to one, leaves
// a NaN remainder: blocks whose results hold a NaN are done again.  A strip with stationary values other than zero below
// 2^-100, above 2^100 or NaN keeps its rows as floats from the start: a bf16 ends at 2^-133 and a third part lies 16 to 17
// binades below its float.  What the parts leave out of streamed values below 2^-110 is then at most d 2^(100 - 134) of a logit.
// (16 x 900 x 128, keys of 2^-122 and queries of 2^122, scores rms against binary64: 2.1e-5 without this rule, 1.7e-7 with
// it.  16 x 1483 x 128 with such a value in every strip: 158 us, 124 without any, 177 when all strips took the fp32 instruction.)
typedef __attribute__((ext_vector_type(4))) uint32_t frag_words;
struct frag_split {
    frag_words w[3];           // as words: selected as eight bf16 they would be taken apart
    __device__ __forceinline__ frag_bf16 p(int n) const { return __builtin_bit_cast(frag_bf16, w[n]); }
};
// The remainders come from the dot instruction of bf16 pairs: a pair of parts by (-1, 0) or (0, -1), added to the float, is one
// instruction where widening the part and subtracting it are two (a whole layer of 16 x 1483 x 128 125 -> 122.5 us, 32 x 2804 x 128
// 572 -> 554).  Exact like the subtraction, subnormal remainders too (the
// tests hold both bit for bit against the host's on 4 million floats of every magnitude); an infinity makes its neighbour in the pair a NaN as well, and so the
// products of that row, which it does without that.
// (The pairs of factors are hidden in registers: from the constant 0x0000bf80 the compiler makes the inline constant
// -1.0, which the instruction takes for 0xbf800000.)
// BOTH: false where `hi` lies past the row (widths of an odd number of steps) and its parts are zeros: from behind those registers
// the compiler does not see that it need not work them out (whole layers, us, subtracted / dots of zeros too / this: 32 x 2804 x 8
// 145.2 / 149.5 / 146.8, x 40 258.9 / 260.4 / 257.4, x 48 282.0 / 287.9 / 282.1; 32 x 5308 x 8 399 / 414 / 401, x 48 806 / 818 / 809).
// DOTS: false for remainders by subtraction, the same bits (see score_kernel in score_any.hip).
template <bool BOTH, bool DOTS>
__device__ __forceinline__ frag_split split_steps(frag_f32 lo, frag_f32 hi)
{
    typedef __attribute__((ext_vector_type(2))) float f2;
    typedef __attribute__((ext_vector_type(2))) __bf16 b2;
    uint32_t first, second;
    asm("s_mov_b32 %0, 0x0000bf80" : "=s"(first));
    asm("s_mov_b32 %0, 0xbf800000" : "=s"(second));
    frag_split s = {};
#pragma unroll
    for (int i = 0; i < (BOTH ? 4 : 2); ++i) {
        f2 x = i < 2 ? f2{lo[2 * i], lo[2 * i + 1]} : f2{hi[2 * i - 4], hi[2 * i - 3]};
#pragma unroll
        for (int part = 0; part < 3; ++part) {
            const b2 b = __builtin_convertvector(x, b2);
            s.w[part][i] = __builtin_bit_cast(uint32_t, b);
            if (part == 2) break;
            if constexpr (DOTS) {
                x[0] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(b2, first), b, x[0], false);
                x[1] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(b2, second), b, x[1], false);
            } else {
                x[0] -= __uint_as_float(s.w[part][i] << 16);
                x[1] -= __uint_as_float(s.w[part][i] & 0xffff0000u);
            }
        }
    }
    return s;
}

// A strip's stationary fragments as the products want them, and the products with a block of 32 streamed rows.
// row(cg) and streamed(rg): this lane's rows of those groups in memory (past the end: any row), for blocks done again and for
// those that in_fp32 (wave-uniform) wants from the fp32 instruction whatever the strip holds.
template <typename T, int KS, int CG> struct frag_strip;
template <int KS, int CG> struct frag_strip<bf16_t, KS, CG> {
    frag_bf16 s[CG][KS];
    __device__ __forceinline__ void set(const frag_bf16 (&f)[CG][KS])
    {
#pragma unroll
        for (int cg = 0; cg < CG; ++cg)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) s[cg][ks] = f[cg][ks];
    }
    template <bool DOTS, typename Row, typename Streamed>
    __device__ __forceinline__ void multiply(const frag_bf16 (&a)[2][KS], acc_t (&acc)[2][CG], int, int, bool, Row&&, Streamed&&) const
    {
#pragma unroll
        for (int cg = 0; cg < CG; ++cg)
#pragma unroll
            for (int rg = 0; rg < 2; ++rg) acc[rg][cg] = acc_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int cg = 0; cg < CG; ++cg)
#pragma unroll
                for (int rg = 0; rg < 2; ++rg) acc[rg][cg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[rg][ks], s[cg][ks], acc[rg][cg], 0, 0, 0);
    }
};
// fp32 with a single group of stationary rows.  Up to 128 dims: strips so few that they do not fill the chip, where a block's
// latency counts and the splitting of its rows only adds to it (2 heads x 256 x 64: 24.3 us the whole layer with bf16 parts, 23.5
// without).  Wider rows, at any number of strips: with one group every streamed row would be split for sixteen stationary
// ones, and two groups of 256 floats in parts take 192 registers beside the streamed 128 (not tried).
template <int KS> struct frag_strip<float, KS, 1> {
    frag_f32 s[KS];
    __device__ __forceinline__ void set(const frag_f32 (&f)[1][KS])
    {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) s[ks] = f[0][ks];
    }
    template <bool DOTS, typename Row, typename Streamed>
    __device__ __forceinline__ void multiply(const frag_f32 (&a)[2][KS], acc_t (&acc)[2][1], int, int, bool, Row&&, Streamed&&) const
    {
#pragma unroll
        for (int rg = 0; rg < 2; ++rg) acc[rg][0] = acc_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int rg = 0; rg < 2; ++rg) acc[rg][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[rg][ks][i], s[ks][i], acc[rg][0], 0, 0, 0);
    }
};
template <int KS, int CG> struct frag_strip<float, KS, CG> {
    static constexpr int KB = (KS + 1) / 2;
    frag_split s[CG][KB];
    bool extreme = false;                      // wave-uniform; the rows are kept as floats then, two steps in the first two parts
    __device__ __forceinline__ void set(const frag_f32 (&f)[CG][KS])
    {
        uint32_t low = ~0u, high = 0;          // twice the bits, without the sign, in `low` less one: a zero comes last
#pragma unroll
        for (int cg = 0; cg < CG; ++cg)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    low = min(low, 2 * __float_as_uint(f[cg][ks][i]) - 1);
                    high = max(high, 2 * __float_as_uint(f[cg][ks][i]));
                }
        extreme = __any(low < 2 * __float_as_uint(0x1p-100f) - 1 || high > 2 * __float_as_uint(0x1p100f));   // (NaN: high)
#pragma unroll
        for (int cg = 0; cg < CG; ++cg)
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                const frag_f32 second = 2 * kb + 1 < KS ? f[cg][(2 * kb + 1) % KS] : frag_f32{};
                if (extreme) {
                    s[cg][kb].w[0] = __builtin_bit_cast(frag_words, f[cg][2 * kb]);
                    s[cg][kb].w[1] = __builtin_bit_cast(frag_words, second);
                    s[cg][kb].w[2] = frag_words{};
                } else {
                    s[cg][kb] = 2 * kb + 1 < KS ? split_steps<true, true>(f[cg][2 * kb], second) : split_steps<false, true>(f[cg][2 * kb], second);
                }
            }
    }
    template <bool DOTS, typename Row, typename Streamed>
    __device__ __forceinline__ void multiply(const frag_f32 (&a)[2][KS], acc_t (&acc)[2][CG], int q4, int d, bool in_fp32, Row&& row, Streamed&& streamed) const
    {
        if (__builtin_expect(extreme, 0)) {    // known beforehand: no parts, and all the rows are in registers
#pragma unroll
            for (int cg = 0; cg < CG; ++cg)
#pragma unroll
                for (int rg = 0; rg < 2; ++rg) acc[rg][cg] = acc_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int cg = 0; cg < CG; ++cg) {
                        const frag_f32 y = __builtin_bit_cast(frag_f32, s[cg][ks / 2].w[ks % 2]);
#pragma unroll
                        for (int rg = 0; rg < 2; ++rg) acc[rg][cg] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[rg][ks][i], y[i], acc[rg][cg], 0, 0, 0);
                    }
            }
            return;
        }
        if (__builtin_expect(!in_fp32, 1)) {
            constexpr int of_a[6] = {0, 2, 1, 0, 1, 0}, of_s[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
            for (int rg = 0; rg < 2; ++rg) {
                frag_split t[KB];
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
                    t[kb] = 2 * kb + 1 < KS ? split_steps<true, DOTS>(a[rg][2 * kb], a[rg][(2 * kb + 1) % KS]) : split_steps<false, DOTS>(a[rg][2 * kb], frag_f32{});
#pragma unroll
                for (int cg = 0; cg < CG; ++cg) acc[rg][cg] = acc_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int n = 0; n < 6; ++n)
#pragma unroll
                    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                        for (int cg = 0; cg < CG; ++cg)
                            acc[rg][cg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(t[kb].p(of_a[n]), s[cg][kb].p(of_s[n]), acc[rg][cg], 0, 0, 0);
            }
            bool nan = false;
#pragma unroll
            for (int cg = 0; cg < CG; ++cg)
#pragma unroll
                for (int rg = 0; rg < 2; ++rg)
                    nan = nan || __builtin_isunordered(acc[rg][cg][0], acc[rg][cg][1]) || __builtin_isunordered(acc[rg][cg][2], acc[rg][cg][3]);
            in_fp32 = __any(nan);
        }
        if (__builtin_expect(in_fp32, 0)) {                              // wave-uniform
#pragma unroll
            for (int cg = 0; cg < CG; ++cg)
#pragma unroll
                for (int rg = 0; rg < 2; ++rg) {
                    const float *x = streamed(rg), *y = row(cg);
                    acc_t c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                    for (int ks = 0; ks < KS; ++ks) {
                        const int at = (ks * 4 + q4) * 4;
                        const frag_f32 u = at < d ? *reinterpret_cast<const frag_f32*>(x + at) : frag_f32{};
                        const frag_f32 w = at < d ? *reinterpret_cast<const frag_f32*>(y + at) : frag_f32{};
#pragma unroll
                        for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(u[i], w[i], c, 0, 0, 0);
                    }
                    acc[rg][cg] = c;
                }
        }
    }
};

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
// stationary rows a wave keeps in registers next to them: as many as 64 registers hold as they are stored (at most 4 groups, 2
// for fp32, whose parts take half as much again: 96 at 128 dims) - or a single group where such strips would leave most of the
// chip idle: strips(rows per strip), fewer than one per compute unit.  The score passes count the strips of
// the query heads for both: with grouped heads pass 2 has fewer workgroups than that, each with several heads to go
// through (32 query heads on 8 key heads x 700 x 64 bf16: 88 for 256 compute units; not tuned).  (All on the fp32
// instruction, a 256-token fp32 prompt of 2 x 64: score passes and matching 21 us with two groups, 16 us with one; 1483 tokens
// of 16 x 128, 750 workgroups: 163 us with two groups, 168 us with one.)
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
