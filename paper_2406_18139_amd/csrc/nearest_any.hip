// Many-to-one nearest-neighbour matching (Section 3.3, Eq. 9): for every evicted key the conserved key with the
// highest cosine similarity, on the ORIGINAL keys - on the matrix cores, for every head width and both types; bf16 with
// head_dim 128 takes the kernels in nearest_mfma.hip.
//
// The L^e x L^c similarity matrix is never stored.  As in score_any.hip a workgroup owns 16 * CG stationary rows - here
// evicted keys, gathered through the evicted list - whose fragments all four waves hold, and the waves share out the
// conserved list: wave w streams the blocks of 32 slots w, w + 4, ... through its own LDS buffer, gathered through the
// conserved list (positions a block ahead of the rows, rows a block ahead of the products).  A lane holds four consecutive
// slots of every 16 against its evicted key and keeps the best value, its slot and the second best value; the sixteen lanes
// that share a key are folded at the end.
// cos(i, j) = (k_i . k_j) * rnorm_i * rnorm_j with rnorm = 1/||k|| (0 for a zero key, which gives cosine 0 against
// everything), compared in fp32.  Ties go to the lower slot.  The matrix instructions add the products of a dot in an order
// of their own.  Where the best values are closer than two orders can bring apart, the dots are added again in the order of
// the dims, a chain of fused multiply-adds, and those values decide: which of several nearly equal keys is matched does
// not hang on the instruction's shape, and a merged row that went to another key would differ visibly.  Two lanes' best
// values are settled by one thread of the key.  Where there may be a third value, or a lane's second, the workgroup goes through
// all the slots of the lanes whose best value is close enough: rare, except among keys that are copies of each other.
// Bound like the score passes by the splitting of the streamed rows (fp32; the vector ALU is busy 52 % of the time at 128 dims and
// 38 % of it is spent waiting) or by the five vector operations per element of the running maxima (bf16, 67 % at 64 dims).
// 922 evicted x 561 conserved keys of 16 x 128 fp32: 30 us (39 on the fp32 instruction, 93 on the vector ALU); 1843 x 938 of
// 32 x 64 bf16: 24 us (126 on the vector ALU; three more with both slots of a lane's best two kept, nine operations); the same
// with some fifteen copies of every image key, so that all keys are looked through again: 280 us (120 us).
#include "frag.h"

#include <type_traits>

namespace lookm {

constexpr int NA_WAVES = 4;

template <typename T>
__global__ void __launch_bounds__(256) k_rnorm(const T* __restrict__ k, size_t rows, int d, float* __restrict__ rnorm)
{
    inverse_norms(k, rows, d, wide_block(), rnorm);
}

// The best two of the lanes' best values and their slots, equal values in the order of their slots, and the largest value
// left over: the third lane's best or a lane's second best.
struct top_two {
    float v1, v2, rest;
    int s1, s2;
    static __device__ __forceinline__ bool before(float av, int as, float bv, int bs) { return av > bv || (av == bv && as < bs); }
    __device__ __forceinline__ void take(float v, int s, float second)
    {
        const bool first = before(v, s, v1, s1), next = before(v, s, v2, s2);
        rest = fmaxf(fmaxf(rest, second), next ? v2 : v);
        v2 = first ? v1 : next ? v : v2;
        s2 = first ? s1 : next ? s : s2;
        v1 = first ? v : v1;
        s1 = first ? s : s1;
    }
};

// A value and its slot as one number, larger for the larger value and then for the lower slot; never zero.
__device__ __forceinline__ unsigned long long pack_value(float v, int slot)
{
    const uint32_t u = __float_as_uint(v);
    return (unsigned long long)(u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u)) << 32 | (uint32_t)~slot;
}

template <typename T, int KS, int CG>
__global__ void __launch_bounds__(256, 2)
k_nearest_any(const T* __restrict__ k, const float* __restrict__ rnorm, const int32_t* __restrict__ kept,
              const int32_t* __restrict__ evicted, int H, int L, int d, int B, int Le, int n_strips,
              int32_t* __restrict__ assign, float* __restrict__ sim)
{
    typedef typename frag<T>::type frag_t;
    constexpr int SR = 16 * CG;
    constexpr int MANY = 4;                          // keys that are looked through again together
    constexpr int BLOCK_BYTES = FRAG_BLOCK * frag_row_bytes<KS>(), FOLD_BYTES = 4 * 3 * SR * 4;
    __shared__ unsigned long long again[SR];
    __shared__ __attribute__((aligned(1024))) char blocks[NA_WAVES][BLOCK_BYTES > FOLD_BYTES ? BLOCK_BYTES : FOLD_BYTES];
    const unsigned unit = wide_block();
    int h, t;                                        // XCD-affine by head, as in k_score_any
    if (H >= 8) {
        const int j = unit >> 3;
        h = (j / n_strips) * 8 + (unit & 7);
        t = j % n_strips;
    } else {
        h = unit % H;
        t = unit / H;
    }
    if (h >= H || t >= n_strips) return;
    k += (size_t)h * L * d;
    rnorm += (size_t)h * L;
    kept += (size_t)h * B;
    evicted += (size_t)h * Le;
    const int e0 = t * SR;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, q4 = lane >> 4, c16 = lane & 15;

    const int n_blocks = (B + 31) / 32;
    char* block = blocks[wave];                      // this wave's conserved rows
    // lane r % 32 holds the position of row r of the block that is fetched next, and the inverse norm of the one in flight
    int pos_next = kept[min(wave * 32 + (lane & 31), B - 1)];
    // Evicted rows: every wave needs all of the strip, loads a quarter into the block buffers and reads all of it.
    frag_strip<T, KS, CG> strip;
    {
        constexpr int RB = frag_row_bytes<KS>(), PART = frag_strip_part<KS, CG>();
        if (wave * PART < SR) {
            const int mine = evicted[min(e0 + wave * PART + (lane & (PART - 1)), Le - 1)];
            frag_load_block<T, KS, PART>(k, d, &blocks[0][0] + wave * PART * RB, lane,
                                         [&](int, int r) { return (uint32_t)__shfl(mine, r) * (uint32_t)(d * sizeof(T)); });
        }
        frag_wait_loads();
        __syncthreads();
        frag_t f[CG][KS];
#pragma unroll
        for (int cg = 0; cg < CG; ++cg) frag_read<T, KS>(&blocks[0][0], cg, c16, q4, d, f[cg]);
        strip.set(f);
        __syncthreads();
    }
    float rn = 0.f;
    auto fetch = [&](int b) {
        rn = rnorm[pos_next];
        if (b * 32 + (lane & 31) >= B) rn = __builtin_nanf("");      // past the end: every comparison with a NaN fails
        const uint32_t row_bytes = (uint32_t)(d * sizeof(T));
        frag_load_block<T, KS, FRAG_BLOCK>(k, d, block, lane, [&](int, int r) { return (uint32_t)__shfl(pos_next, r) * row_bytes; });
        pos_next = kept[min((b + NA_WAVES) * 32 + (lane & 31), B - 1)];
    };
    float v1[CG], v2[CG];
    int s1[CG];
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) { v1[cg] = v2[cg] = -INFINITY; s1[cg] = 0x7fffffff; }
    if (wave < n_blocks) fetch(wave);
    for (int b = wave; b < n_blocks; b += NA_WAVES) {
        frag_wait_loads();
        asm volatile("" ::: "memory");
        frag_t a[2][KS];
        float r[2][4];
#pragma unroll
        for (int rg = 0; rg < 2; ++rg) {
            frag_read<T, KS>(block, rg, c16, q4, d, a[rg]);
#pragma unroll
            for (int i = 0; i < 4; ++i) r[rg][i] = __shfl(rn, 16 * rg + 4 * q4 + i);
        }
        const bool tiny = sizeof(T) == 4 && __any(rn > 0x1p100f);    // a conserved row too short for bf16 parts to give its direction
        __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): the fragments are in registers, the block may be refilled
        __builtin_amdgcn_sched_barrier(0);
        if (b + NA_WAVES < n_blocks) fetch(b + NA_WAVES);
        __builtin_amdgcn_sched_barrier(0);
        acc_t acc[2][CG];
        strip.template multiply<true>(a, acc, q4, d, tiny, [&](int cg) { return k + (size_t)evicted[min(e0 + 16 * cg + c16, Le - 1)] * d; },
                       [&](int rg) { return k + (size_t)kept[min(b * 32 + 16 * rg + c16, B - 1)] * d; });
#pragma unroll
        for (int cg = 0; cg < CG; ++cg)
#pragma unroll
            for (int rg = 0; rg < 2; ++rg)
#pragma unroll
                for (int i = 0; i < 4; ++i) {                         // ascending slot inside the lane
                    const float v = acc[rg][cg][i] * r[rg][i];
                    const int s = b * 32 + 16 * rg + 4 * q4 + i;
                    const bool first = v > v1[cg];
                    v2[cg] = __builtin_amdgcn_fmed3f(v, v1[cg], v2[cg]);    // (with a NaN the smaller of the others)
                    v1[cg] = first ? v : v1[cg];
                    s1[cg] = first ? s : s1[cg];
                }
    }

    // [wave][lane's q4][key] best values, second best values, slots, in place of the waves' blocks
    auto fold_v = [&](int j, int what) { return reinterpret_cast<float*>(blocks[j >> 2]) + (what * 4 + (j & 3)) * SR; };
    auto fold_s = [&](int j) { return reinterpret_cast<int*>(blocks[j >> 2]) + (8 + (j & 3)) * SR; };
    constexpr int LANES = NA_WAVES * 4;              // that share a key
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) {
        fold_v(wave * 4 + q4, 0)[16 * cg + c16] = v1[cg];
        fold_v(wave * 4 + q4, 1)[16 * cg + c16] = v2[cg];
        fold_s(wave * 4 + q4)[16 * cg + c16] = s1[cg];
    }
    if (tid < SR) again[tid] = 0;
    // every wave folds the sixteen lanes of evicted key e0 + lane; a strip of fewer than 64 keys shares them out to the lanes
    const bool mine = lane < SR && e0 + lane < Le;
    const int at = min(lane % SR, Le - 1 - e0);
    const int e_row = evicted[e0 + at];
    const float e_rn = rnorm[e_row];
    __syncthreads();
    top_two found{-INFINITY, -INFINITY, -INFINITY, 0x7fffffff, 0x7fffffff};
#pragma unroll
    for (int i = 0; i < LANES; i += 64 / SR) {
        const int j = i + lane / SR;
        found.take(fold_v(j, 0)[at], fold_s(j)[at], fold_v(j, 1)[at]);
    }
#pragma unroll
    for (int step = SR; step < 64; step <<= 1) {
        const top_two o{__shfl_xor(found.v1, step), __shfl_xor(found.v2, step), __shfl_xor(found.rest, step),
                        __shfl_xor(found.s1, step), __shfl_xor(found.s2, step)};
        found.take(o.v1, o.s1, o.rest);
        found.take(o.v2, o.s2, -INFINITY);
    }
    float v = found.v1;
    int s = found.s1;
    // A sum of d products in any order, roundings to nearest or towards zero, is off by at most d 2^-23 |e| |c|, the chain of fused
    // multiply-adds by half of that, and the factor 1 / |c| adds a rounding to each: two values that the other order can swap
    // are within 6 (d + 1) 2^-24 |e| of each other (|e| = 1 / e_rn).  fp32 products from bf16 parts leave out less than 2^-24 |e| |c| and
    // add up their small parts, five times d terms of at most 2^-7 |e| |c| together, first: (7 d + 8) 2^-24.  A key of norm zero has all values zero in every order.
    // A bound, not an estimate: with d = 64 it sends a few keys in a hundred to the second look, and about one in a thousand
    // because of a third value (or of two in one lane) through a sixteenth of the slots or a few.
    const float band = (sizeof(T) == 4 ? 7.f * (float)d + 8.f : 6.f * (float)(d + 1)) * 0x1p-24f;
    auto close = [&](float x) { return (found.v1 - x) * e_rn <= band; };
    const uint64_t many = __ballot(mine && found.s1 < B && e_rn != 0.f && close(found.rest));      // alike in all four waves
    if (wave == 0 && mine && found.s2 < B && close(found.v2) && !((many >> lane) & 1)) {
        const int c1 = kept[found.s1], c2 = kept[found.s2];
        const T *ke = k + (size_t)e_row * d, *k1 = k + (size_t)c1 * d, *k2 = k + (size_t)c2 * d;
        float d1 = 0.f, d2 = 0.f;
#pragma unroll sizeof(T) == 2 ? 4 : 2     // (fp32: four would take more registers than the products)
        for (int c = 0; c < d; c += 8) {
            float xe[8], x1[8], x2[8];
            load8(ke + c, xe);
            load8(k1 + c, x1);
            load8(k2 + c, x2);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                d1 = fmaf(xe[i], x1[i], d1);
                d2 = fmaf(xe[i], x2[i], d2);
            }
        }
        d1 *= rnorm[c1];
        d2 *= rnorm[c2];
        const bool other = top_two::before(d2, found.s2, d1, found.s1);
        v = other ? d2 : d1;
        s = other ? found.s2 : found.s1;
    }
    if (__builtin_expect(many != 0, 0)) {
        unsigned lanes = 0;                          // those whose best value may not be this key's best
#pragma unroll
        for (int j = 0; j < LANES; ++j) lanes |= close(fold_v(j, 0)[at]) ? 1u << j : 0u;
        const float least = found.v1 - band / e_rn;  // no smaller value can be the best
        float* rows = reinterpret_cast<float*>(blocks[0]);     // the keys in hand, in fp32
        const int per_lane = (n_blocks + NA_WAVES - 1) / NA_WAVES * 8;
        for (uint64_t todo = many; todo != 0;) {
            int r[MANY], row[MANY];
            float low[MANY];
            unsigned seen = 0;
#pragma unroll
            for (int n = 0; n < MANY; ++n) {         // fewer left: the last one again
                r[n] = (n == 0 || todo != 0) ? __builtin_ctzll(todo) : r[n > 0 ? n - 1 : 0];
                row[n] = __builtin_amdgcn_readlane(e_row, r[n]);
                low[n] = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(least), r[n]));
                seen |= (unsigned)__builtin_amdgcn_readlane((int)lanes, r[n]);
                todo &= todo - 1;
            }
            __syncthreads();                         // all waves have read what lies in the blocks
#pragma unroll
            for (int n = 0; n < MANY; ++n)
                if (wave == n % NA_WAVES && lane * 8 < d) {
                    float y[8];
                    load8(k + (size_t)row[n] * d + lane * 8, y);
                    store8(rows + n * d + lane * 8, y);
                }
            __syncthreads();
            for (int x = tid; x < __popc(seen) * per_lane; x += 64 * NA_WAVES) {
                unsigned left = seen;
                for (int skip = x / per_lane; skip > 0; --skip) left &= left - 1;
                const int j = __builtin_ctz(left), y = x % per_lane;
                const int slot = ((j >> 2) + NA_WAVES * (y >> 3)) * 32 + ((y >> 2) & 1) * 16 + (j & 3) * 4 + (y & 3);
                if (slot >= B) continue;
                const int pos = kept[slot];
                const T* kc = k + (size_t)pos * d;
                float dot[MANY] = {};
#pragma unroll 4
                for (int c = 0; c < d; c += 8) {     // every key's sum in the order of the dims
                    float xc[8], ye[8];
                    load8(kc + c, xc);
#pragma unroll
                    for (int n = 0; n < MANY; ++n) {
                        load8(rows + n * d + c, ye);
#pragma unroll
                        for (int i = 0; i < 8; ++i) dot[n] = fmaf(ye[i], xc[i], dot[n]);
                    }
                }
                const float rn = rnorm[pos];
#pragma unroll
                for (int n = 0; n < MANY; ++n)
                    if (dot[n] * rn >= low[n]) atomicMax(&again[r[n]], pack_value(dot[n] * rn, slot));
            }
        }
        __syncthreads();
        if (((many >> lane) & 1) && again[at] != 0) {
            const uint32_t u = (uint32_t)(again[at] >> 32);
            v = __uint_as_float(u ^ ((u >> 31) ? 0x80000000u : 0xffffffffu));
            s = (int)~(uint32_t)again[at];
        }
    }
    if (wave == 0 && mine) {
        const size_t e = (size_t)h * Le + e0 + lane;
        assign[e] = s;
        sim[e] = v * e_rn;
    }
}

}  // namespace lookm

namespace lookm_host {

int launch_nearest_mfma(const void* k, const int32_t* kept, const int32_t* evicted, int H, int L, int budget,
                        const float* rnorm, int32_t* assign, float* sim, void* scratch, hipStream_t st);
size_t nearest_mfma_scratch_bytes(int H, int L, int B);

template <typename T>
static int launch_nearest_t(const T* k, const int32_t* kept, const int32_t* evicted, int H, int L, int d, int budget,
                            float* rnorm, bool rnorm_ready, int32_t* assign, float* sim, void* scratch, hipStream_t st,
                            bool mfma)
{
    const int Le = L - budget;
    if (Le == 0) return LOOKM_OK;
    const LaunchCheck check;
    const size_t rows = (size_t)H * L;
    if (!rnorm_ready)
        hipLaunchKernelGGL(lookm::k_rnorm<T>, wide_grid((rows + 31) / 32), dim3(256), 0, st, k, rows, d, rnorm);
    mark(LOOKM_K_RNORM);
    if (mfma) return launch_nearest_mfma(k, kept, evicted, H, L, budget, rnorm, assign, sim, scratch, st);
    lookm::with_frag_shape<T>(d, [&](int rows) { return (long)((Le + rows - 1) / rows) * H; }, [&](auto steps, auto groups) {
        constexpr int KS = decltype(steps)::value, CG = decltype(groups)::value;
        const int strips = (Le + 16 * CG - 1) / (16 * CG);
        hipLaunchKernelGGL((lookm::k_nearest_any<T, KS, CG>), wide_grid((size_t)(H >= 8 ? (H + 7) / 8 * 8 : H) * strips), dim3(256), 0, st,
                           k, rnorm, kept, evicted, H, L, d, budget, Le, strips, assign, sim);
    });
    mark(LOOKM_K_NEAREST);
    return check.status();
}

size_t nearest_scratch_bytes(int H, int L, int d, lookm_dtype dt, int budget)
{
    return (dt == LOOKM_BF16 && d == 128) ? nearest_mfma_scratch_bytes(H, L, budget) : 0;
}

int launch_nearest(const void* k, const int32_t* kept, const int32_t* evicted, int H, int L, int d, lookm_dtype dt,
                   int budget, float* rnorm, bool rnorm_ready, int32_t* assign, float* sim, void* scratch,
                   hipStream_t st)
{
    if (dt == LOOKM_BF16)
        return launch_nearest_t((const lookm::bf16_t*)k, kept, evicted, H, L, d, budget, rnorm, rnorm_ready, assign,
                                sim, scratch, st, d == 128);
    return launch_nearest_t((const float*)k, kept, evicted, H, L, d, budget, rnorm, rnorm_ready, assign, sim, scratch,
                            st, false);
}

}  // namespace lookm_host
