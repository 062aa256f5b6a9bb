// Many-to-one nearest-neighbour matching (Section 3.3, Eq. 9): for every evicted key the conserved key with the
// highest cosine similarity, on the ORIGINAL keys - on the matrix cores, for every head width and both types; bf16 with
// head_dim 128 takes the kernels in nearest_mfma.hip.
//
// The L^e x L^c similarity matrix is never stored.  As in score_any.hip a workgroup owns 16 * CG stationary rows - here
// evicted keys, gathered through the evicted list - whose fragments all four waves hold, and the waves share out the
// conserved list: wave w streams the blocks of 32 slots w, w + 4, ... through its own LDS buffer, gathered through the
// conserved list (positions a block ahead of the rows, rows a block ahead of the products).  A lane holds four consecutive
// slots of every 16 against its evicted key and keeps the two best values and their slots; the four lanes of a key and then
// the four waves are folded at the end.
// cos(i, j) = (k_i . k_j) * rnorm_i * rnorm_j with rnorm = 1/||k|| (0 for a zero key, which gives cosine 0 against
// everything), compared in fp32.  Ties go to the lower slot.  The matrix instructions add the products of a dot in an order
// of their own.  Where the two best values are closer than two orders can bring apart, one thread per key adds both dots in
// the order of the dims, a chain of fused multiply-adds, and those values decide: which of two nearly equal keys is
// matched does not hang on the instruction's shape, and a merged row that went to another key would differ visibly.
// Bound like the score passes, by the fp32 matrix instruction or (bf16) by the nine vector operations per element of
// the two running maxima.  922 evicted x 561 conserved keys of 16 x 128 fp32: 37 us (on the vector ALU: 85 us); 1843 x 938
// of 32 x 64 bf16: 30 us (110 us); with the best value alone, four operations and no second look, 35 and 21 us.  The second
// value by a median instruction instead of two selects: no faster.
#include "frag.h"

#include <type_traits>

namespace lookm {

constexpr int NA_WAVES = 4;

template <typename T>
__global__ void __launch_bounds__(256) k_rnorm(const T* __restrict__ k, size_t rows, int d, float* __restrict__ rnorm)
{
    inverse_norms(k, rows, d, wide_block(), rnorm);
}

// The best and the second best value and their slots; equal values in the order of their slots.
struct top_two {
    float v1, v2;
    int s1, s2;
    static __device__ __forceinline__ bool before(float av, int as, float bv, int bs) { return av > bv || (av == bv && as < bs); }
    __device__ __forceinline__ void take(const top_two& o)
    {
        if (before(o.v1, o.s1, v1, s1)) {
            if (before(o.v2, o.s2, v1, s1)) { v2 = o.v2; s2 = o.s2; }
            else { v2 = v1; s2 = s1; }
            v1 = o.v1;
            s1 = o.s1;
        } else if (before(o.v1, o.s1, v2, s2)) {
            v2 = o.v1;
            s2 = o.s1;
        }
    }
};

template <typename T, int KS, int CG>
__global__ void __launch_bounds__(256, 2)
k_nearest_any(const T* __restrict__ k, const float* __restrict__ rnorm, const int32_t* __restrict__ kept,
              const int32_t* __restrict__ evicted, int H, int L, int d, int B, int Le, int n_strips,
              int32_t* __restrict__ assign, float* __restrict__ sim)
{
    typedef typename frag<T>::type frag_t;
    constexpr int SR = 16 * CG;
    __shared__ top_two fold[NA_WAVES][SR];
    __shared__ __attribute__((aligned(1024))) char blocks[NA_WAVES][FRAG_BLOCK * frag_row_bytes<KS>()];
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
    frag_t sf[CG][KS];
#pragma unroll
    for (int cg = 0; cg < CG; ++cg)
        frag_stationary<T, KS>(k + (size_t)evicted[min(e0 + 16 * cg + c16, Le - 1)] * d, q4, d, sf[cg]);

    // lane r % 32 holds the position of row r of the block that is fetched next, and the inverse norm of the one in flight
    int pos_next = kept[min(wave * 32 + (lane & 31), B - 1)];
    float rn = 0.f;
    auto fetch = [&](int b) {
        rn = rnorm[pos_next];
        if (b * 32 + (lane & 31) >= B) rn = __builtin_nanf("");      // past the end: every comparison with a NaN fails
        const uint32_t row_bytes = (uint32_t)(d * sizeof(T));
        frag_load_block<T, KS>(k, d, block, lane, [&](int, int r) { return (uint32_t)__shfl(pos_next, r) * row_bytes; });
        pos_next = kept[min((b + NA_WAVES) * 32 + (lane & 31), B - 1)];
    };
    top_two top[CG];
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) top[cg] = top_two{-INFINITY, -INFINITY, 0x7fffffff, 0x7fffffff};
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
        __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): the fragments are in registers, the block may be refilled
        __builtin_amdgcn_sched_barrier(0);
        if (b + NA_WAVES < n_blocks) fetch(b + NA_WAVES);
        __builtin_amdgcn_sched_barrier(0);
        acc_t acc[2][CG];
#pragma unroll
        for (int cg = 0; cg < CG; ++cg)
#pragma unroll
            for (int rg = 0; rg < 2; ++rg) acc[rg][cg] = acc_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int i = 0; i < frag<T>::SUB; ++i)
#pragma unroll
                for (int cg = 0; cg < CG; ++cg)
#pragma unroll
                    for (int rg = 0; rg < 2; ++rg) acc[rg][cg] = frag<T>::mma(i, a[rg][ks], sf[cg][ks], acc[rg][cg]);
#pragma unroll
        for (int cg = 0; cg < CG; ++cg)
#pragma unroll
            for (int rg = 0; rg < 2; ++rg)
#pragma unroll
                for (int i = 0; i < 4; ++i) {                         // ascending slot inside the lane
                    const float v = acc[rg][cg][i] * r[rg][i];
                    const int s = b * 32 + 16 * rg + 4 * q4 + i;
                    top_two& t = top[cg];
                    const bool first = v > t.v1, second = v > t.v2;
                    t.v2 = first ? t.v1 : second ? v : t.v2;
                    t.s2 = first ? t.s1 : second ? s : t.s2;
                    t.v1 = first ? v : t.v1;
                    t.s1 = first ? s : t.s1;
                }
    }

#pragma unroll
    for (int cg = 0; cg < CG; ++cg) {
#pragma unroll
        for (int step = 16; step <= 32; step <<= 1)
            top[cg].take(top_two{__shfl_xor(top[cg].v1, step), __shfl_xor(top[cg].v2, step), __shfl_xor(top[cg].s1, step),
                                 __shfl_xor(top[cg].s2, step)});
        if (q4 == 0) fold[wave][16 * cg + c16] = top[cg];
    }
    __syncthreads();
    if (tid < SR && e0 + tid < Le) {
        top_two t = fold[0][tid];
#pragma unroll
        for (int w = 1; w < NA_WAVES; ++w) t.take(fold[w][tid]);
        const int e_row = evicted[e0 + tid];
        const float e_rn = rnorm[e_row];
        float v = t.v1;
        int s = t.s1;
        // Any order of the sum of a dot is off by at most d 2^-24 |e| |c|, and the factor 1 / |c| adds one rounding: two
        // values that another order can swap are within 4 (d + 1) 2^-24 |e| of each other (|e| = 1 / e_rn; a key of norm
        // zero has all values zero).  A bound, not an estimate: with d = 64 it sends a few keys in a hundred here.
        if (t.s2 < B && (t.v1 - t.v2) * e_rn <= 4.f * (float)(d + 1) * 0x1p-24f) {
            const int c1 = kept[t.s1], c2 = kept[t.s2];
            const T *ke = k + (size_t)e_row * d, *k1 = k + (size_t)c1 * d, *k2 = k + (size_t)c2 * d;
            float d1 = 0.f, d2 = 0.f;
#pragma unroll 4
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
            const bool other = top_two::before(d2, t.s2, d1, t.s1);
            v = other ? d2 : d1;
            s = other ? t.s2 : t.s1;
        }
        const size_t e = (size_t)h * Le + e0 + tid;
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
