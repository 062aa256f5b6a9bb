// Accumulated attention scores (Section 3.2, Eq. 4) on the gfx950 matrix cores for every head width and both types;
// bf16 with 128-wide heads takes the LDS-tiled kernels in score_mfma.hip.
//
// Two passes over the causal half of Q K^T, neither of which stores it:
//   pass 1: lse2[i] = log2 sum_{j<=i} 2^(c * q_i.k_j),  c = log2(e)/sqrt(d)
//   pass 2: A_s[j]  = sum_{i>=j} 2^(c * q_i.k_j - lse2[i])
// A workgroup owns 16 * CG stationary rows - query rows in pass 1, keys in pass 2 - whose operand fragments every one
// of its four waves keeps in registers, and the waves share out the other axis: wave w streams the 32-row blocks w,
// w + 4, ... through its own LDS buffer (see frag.h), the next block on its way during the current block's products.
// No barrier in the loop.  Of a 16x16 tile, lane (c, q) holds the streamed rows 4q .. 4q+3 against stationary row c,
// so both reductions are in-lane; the four lanes of a row and then the four waves are folded once at the end, in a
// fixed order.  Splitting the streamed axis over the waves of one workgroup, instead of over workgroups with a fold
// kernel behind them, leaves short strips (64 rows; 32 or 16 in fp32), so that a few hundred tokens already make
// enough workgroups, and nothing is written but the result.
//
// What bounds it: bf16 - the vector ALU, busy 80 % of the time in pass 1 and 75 % in pass 2 at 64 dims with an exponential and its
// two companions per logit.  fp32 - the splitting of every streamed row into bf16 parts for every strip (three and
// a half instructions a float, two of them dots): at 64 dims and four waves a SIMD the vector
// ALU is busy 66 % (pass 1) and the matrix pipe 44 %, one or both all the time; at 128, two waves, 50 % and 36 %, one or both
// 81 % (dots leave the matrix pipe less company: both at once 13 % of its time, with subtractions 31 %), and the longest strips run alone for the last fifth.  Both passes, traced:
// 16 heads x 1483 x 128 fp32 84 us (126 on the fp32 matrix instruction, beside which the vector ALU stands
// still; 685 on the vector ALU, with 64 x 64 tiles in LDS), 32 x 2781 x 64 bf16 60 us (790), x 80 74 us, 2 x 256 x 64 fp32
// 10 us (64).  Stationary rows through LDS, blocks through a buffer descriptor, log-sum-exps straight to LDS and the first block
// of a wave without a sum against a reference that it has not got, all timed with events: 121 -> 105 us for the first (on the
// fp32 instruction), 62 -> 55 for the second.
// (Tried: every other 32 workgroups of an XCD in the opposite order, so that long strips meet short ones on a compute unit:
// no gain, the third lot undoes it; fp32 blocks of 16 rows, three workgroups a compute unit: pass 1 52 -> 56 us.)
#include "frag.h"

#include <algorithm>
#include <type_traits>

namespace lookm {

constexpr int SA_WAVES = 4;

// sum over a block of 32 streamed keys against the reference of each row; a row whose sum overflows gets a new
// reference, and a NaN reaches the sum either way (see score_mfma.hip)
template <int CG>
__device__ __forceinline__ void lse_update(const acc_t (&acc)[2][CG], float scale2, float (&m)[CG], float (&l)[CG], bool first)
{
    float sum[CG], top = INFINITY;
    if (!first)             // (scalar; a wave's first block has no reference yet)
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) {
#pragma unroll
        for (int rg = 0; rg < 2; ++rg)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float p = __builtin_amdgcn_exp2f(fmaf(acc[rg][cg][i], scale2, -m[cg]));
                sum[cg] = (rg == 0 && i == 0) ? p : sum[cg] + p;
            }
        top = (cg == 0) ? sum[cg] : fmaxf(top, sum[cg]);
    }
    if (__builtin_expect(__any(top > 1.8e19f), 0)) {
#pragma unroll
        for (int cg = 0; cg < CG; ++cg) {
            float bm = acc[0][cg][0];
#pragma unroll
            for (int i = 1; i < 8; ++i) bm = fmaxf(bm, acc[i >> 2][cg][i & 3]);
            const float mn = fmaxf(m[cg], bm * scale2);
            float s = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) s += __builtin_amdgcn_exp2f(fmaf(acc[i >> 2][cg][i & 3], scale2, -mn));
            l[cg] = fmaf(l[cg], __builtin_amdgcn_exp2f(m[cg] - mn), s);
            m[cg] = mn;
            sum[cg] = 0.f;     // in l already, with one rounding
        }
    }
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) l[cg] += sum[cg];
}

// This thread's share of the sums over FEW keys of one query head, rows thread, thread + 256, ... from each key on: dots in
// the order of the dims on the vector ALU and exp2f, which gives weights down to 2^-149.
constexpr int FEW = 4;
template <typename T>
__device__ __forceinline__ void weights_of_keys(const T* __restrict__ q, const T* __restrict__ k, const float* __restrict__ lse2,
                                                const int (&key)[FEW], int R0, int L, int d, float scale2, float lse_scale,
                                                float (&sum)[FEW])
{
    for (int i = max(key[0], R0) + (int)threadIdx.x; i < L; i += 64 * SA_WAVES) {        // key[0] is the lowest
        float dot[FEW] = {};
#pragma unroll sizeof(T) == 2 ? 2 : 1      // (fp32: two steps of four keys take more scalar registers than there are)
        for (int c = 0; c < d; c += 8) {
            float y[8];
            load8(q + (size_t)i * d + c, y);
#pragma unroll
            for (int n = 0; n < FEW; ++n) {
                float x[8];
                load8(k + (size_t)key[n] * d + c, x);
#pragma unroll
                for (int e = 0; e < 8; ++e) dot[n] = fmaf(y[e], x[e], dot[n]);
            }
        }
        const float neg = -lse2[i] * lse_scale;
#pragma unroll
        for (int n = 0; n < FEW; ++n) {
            const float p = exp2f(fmaf(dot[n], scale2, neg));
            sum[n] += (i >= key[n]) ? p : 0.f;
        }
    }
}

// PASS 1: stationary q (query heads), streamed k; writes lse2.  PASS 2: stationary k (key heads), streamed q of each of
// the `group` query heads in turn; writes scores.  Workgroups from n_units on compute the inverse norms of norm_rows keys.
// MODE: the pass, and SUBTRACT where the remainders of fp32 parts are differences instead of dots.
constexpr int SUBTRACT = 4;
template <int MODE, typename T, int KS, int CG>
__global__ void __launch_bounds__(256, 2)
k_score_any(const T* __restrict__ q, const T* __restrict__ k, int heads, int group, int L, int R0, int d, float scale2,
            const float* __restrict__ lse2, float lse_scale, float* __restrict__ out, int n_strips, int together, unsigned n_units,
            size_t norm_rows, float* __restrict__ rnorm)
{
    constexpr int PASS = MODE % SUBTRACT;
    typedef typename frag<T>::type frag_t;
    constexpr int SR = 16 * CG;                      // stationary rows
    __shared__ float fold_a[SA_WAVES][SR], fold_b[PASS == 1 ? SA_WAVES : 1][SR];
    __shared__ __attribute__((aligned(1024))) char blocks[SA_WAVES][FRAG_BLOCK * frag_row_bytes<KS>()];
    __shared__ __attribute__((aligned(256))) float refs[PASS == 2 ? SA_WAVES : 1][64];
    const unsigned unit = wide_block();
    if (unit >= n_units) {
        inverse_norms(k, norm_rows, d, unit - n_units, rnorm);
        return;
    }
    // consecutive workgroups go to consecutive XCDs: with eight or more heads XCD x works through the heads x, x + 8, ...,
    // `together` of them at a time (as many as its L2 holds the streamed rows of), the longest strips of those first
    int h, t;
    if (heads >= 8) {
        const int j = unit >> 3, set = j / (n_strips * together), in_set = j % (n_strips * together);
        const int n = min(together, (heads + 7) / 8 - set * together);         // heads in this set
        h = (set * together + in_set % n) * 8 + (unit & 7);
        t = in_set / n;
    } else {
        h = unit % heads;
        t = unit / heads;
    }
    if (h >= heads) return;
    const int nS = (L + SR - 1) / SR;
    const int s0 = ((PASS == 1) ? nS - 1 - t : t) * SR;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, q4 = lane >> 4, c16 = lane & 15;
    char* block = blocks[wave];                     // this wave's streamed block

    const T* S = (PASS == 1) ? q + (size_t)h * L * d : k + (size_t)h * L * d;
    int off[frag_row_kinds<KS>()];
    frag_row_offsets<T, KS>(d, lane, off);
    // Stationary rows: every wave needs all of them, so each loads a quarter of the strip - into the buffers that the
    // streamed blocks take afterwards - and reads all of it.  (Fragments straight from global memory touch sixteen cache
    // lines for 1 KB: 3 us of a compute unit's L1 for its 128 KB.)
    frag_strip<T, KS, CG> strip;
    {
        constexpr int RB = frag_row_bytes<KS>(), PART = frag_strip_part<KS, CG>();
        const auto srsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(S), 0, L * d * (int)sizeof(T), 0x00020000);
        if (wave * PART < SR)
            frag_load_rows<T, KS, PART>(srsrc, d, &blocks[0][0] + wave * PART * RB, lane, off, min(s0 + wave * PART, L - 1), L - min(s0 + wave * PART, L - 1));
        frag_wait_loads();
        __syncthreads();
        frag_t f[CG][KS];
#pragma unroll
        for (int cg = 0; cg < CG; ++cg) frag_read<T, KS>(&blocks[0][0], cg, c16, q4, d, f[cg]);
        strip.set(f);
        __syncthreads();
    }

    float m[CG], l[CG];                              // pass 1: reference and sum per stationary row; pass 2: l only
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) { m[cg] = -1e30f; l[cg] = 0.f; }

    // streamed rows [b0 * 32, x_end) in blocks of 32
    const int x_end = (PASS == 1) ? min(L, s0 + SR) : L;
    const int b0 = ((PASS == 1) ? 0 : max(s0, R0)) / 32 + wave, b_end = (x_end + 31) / 32;
    const int n_heads = (PASS == 1) ? 1 : group;
    for (int g = 0; g < n_heads; ++g) {
        const T* X = (PASS == 1) ? k + (size_t)(h / group) * L * d : q + ((size_t)h * group + g) * L * d;
        const float* lse_h = lse2 + ((size_t)h * group + g) * L;        // pass 2
        const auto xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(X), 0, L * d * (int)sizeof(T), 0x00020000);
        frag_t a[2][KS];
        auto fetch = [&](int b) {
            if (PASS == 2) {                                           // log-sum-exp of the block's rows (and of 32 more)
                const int row = (b * 32 + 64 <= L) ? b * 32 + lane : min(b * 32 + lane, L - 1);
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(lse_h + row),
                                                 (__attribute__((address_space(3))) void*)refs[PASS == 2 ? wave : 0], 4, 0, 0);
            }
            frag_load_rows<T, KS, FRAG_BLOCK>(xrsrc, d, block, lane, off, b * 32, L - b * 32);
        };
        if (b0 < b_end) fetch(b0);
        for (int b = b0; b < b_end; b += SA_WAVES) {
            frag_wait_loads();
            asm volatile("" ::: "memory");
#pragma unroll
            for (int rg = 0; rg < 2; ++rg) frag_read<T, KS>(block, rg, c16, q4, d, a[rg]);
            float neg[2][4];                         // pass 2: -log-sum-exp of the lane's eight streamed rows
            if (PASS == 2)
#pragma unroll
                for (int rg = 0; rg < 2; ++rg) {
                    const float4 v = *reinterpret_cast<const float4*>(&refs[PASS == 2 ? wave : 0][16 * rg + 4 * q4]);
                    neg[rg][0] = -v.x * lse_scale;
                    neg[rg][1] = -v.y * lse_scale;
                    neg[rg][2] = -v.z * lse_scale;
                    neg[rg][3] = -v.w * lse_scale;
                }
            // the block is in registers: the next one's rows may take its place in LDS
            __builtin_amdgcn_s_waitcnt(0xC07F);      // lgkmcnt(0): the fragments have arrived
            __builtin_amdgcn_sched_barrier(0);
            if (b + SA_WAVES < b_end) fetch(b + SA_WAVES);
            __builtin_amdgcn_sched_barrier(0);
            acc_t acc[2][CG];
            strip.template multiply<MODE < SUBTRACT>(a, acc, q4, d, false, [&](int cg) { return S + (size_t)min(s0 + 16 * cg + c16, L - 1) * d; },
                           [&](int rg) { return X + (size_t)min(b * 32 + 16 * rg + c16, L - 1) * d; });
            const int xq = b * 32 + 4 * q4;          // streamed row of entry i of acc[rg][.]: xq + 16*rg + i
            if (PASS == 1) {
                if (b * 32 + 31 > s0) {              // blocks on the diagonal are masked element by element (wave-uniform)
#pragma unroll
                    for (int cg = 0; cg < CG; ++cg)
#pragma unroll
                        for (int rg = 0; rg < 2; ++rg)
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                if (xq + 16 * rg + i > s0 + 16 * cg + c16) acc[rg][cg][i] = -INFINITY;   // key after the query
                }
                lse_update<CG>(acc, scale2, m, l, b == b0);
            } else {
                // masked: terms of rows before the key, before the observation window and past the end are not added at all (as
                // -inf in the exponent they would still meet the row's log-sum-exp, which may be infinite or NaN)
                const bool masked = b * 32 < max(s0 + SR - 1, R0) || b * 32 + 32 > L;       // scalar
                float p[2][CG][4];
#pragma unroll
                for (int cg = 0; cg < CG; ++cg)
#pragma unroll
                    for (int rg = 0; rg < 2; ++rg)
#pragma unroll
                        for (int i = 0; i < 4; ++i) p[rg][cg][i] = __builtin_amdgcn_exp2f(fmaf(acc[rg][cg][i], scale2, neg[rg][i]));
                if (masked)
#pragma unroll
                    for (int cg = 0; cg < CG; ++cg)
#pragma unroll
                        for (int rg = 0; rg < 2; ++rg)
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const int x = xq + 16 * rg + i;
                                if (x < max(s0 + 16 * cg + c16, R0) || x >= L) p[rg][cg][i] = 0.f;
                            }
#pragma unroll
                for (int cg = 0; cg < CG; ++cg) {
                    float sum = 0.f;
#pragma unroll
                    for (int rg = 0; rg < 2; ++rg)
#pragma unroll
                        for (int i = 0; i < 4; ++i) sum = (rg == 0 && i == 0) ? p[rg][cg][i] : sum + p[rg][cg][i];
                    l[cg] += sum;
                }
            }
        }
    }

    // fold the four lanes of a stationary row, then the waves in order
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) {
#pragma unroll
        for (int step = 16; step <= 32; step <<= 1) {          // (only the lower lane of a pair is read from here on)
            const float lo = __shfl_xor(l[cg], step);
            if (PASS == 1) {
                const float mo = __shfl_xor(m[cg], step), M = fmaxf(m[cg], mo);
                l[cg] = l[cg] * __builtin_amdgcn_exp2f(m[cg] - M) + lo * __builtin_amdgcn_exp2f(mo - M);
                m[cg] = M;
            } else {
                l[cg] += lo;
            }
        }
        if (q4 == 0) {
            fold_a[wave][16 * cg + c16] = l[cg];
            if (PASS == 1) fold_b[PASS == 1 ? wave : 0][16 * cg + c16] = m[cg];
        }
    }
    __syncthreads();
    const bool mine = lane < SR && s0 + lane < L;    // every wave folds the waves' sums: row s0 + lane
    float sum = 0.f;
    if (PASS == 1) {
        if (wave != 0 || !mine) return;
        float M = -1e30f;
#pragma unroll
        for (int w = 0; w < SA_WAVES; ++w) M = fmaxf(M, fold_b[PASS == 1 ? w : 0][lane]);
#pragma unroll
        for (int w = 0; w < SA_WAVES; ++w) sum = fmaf(fold_a[w][lane], exp2f(fold_b[PASS == 1 ? w : 0][lane] - M), sum);
        sum = M + log2f(sum);
    } else {
        auto fold = [&]() {
            float f = 0.f;
#pragma unroll
            for (int w = 0; w < SA_WAVES; ++w) f += fold_a[w][lane];
            return f;
        };
        if (mine) sum = fold();
        // The bare exponential instruction gives zero for weights below 2^-126.  `n` of them are below n * 2^-126: a sum above
        // n * 2^-102 has lost nothing in its 24 bits, a smaller one is worked out again with exp2f, which gives subnormal
        // weights too, so that keys that hardly any query looks at are still told apart.  (exp2f in the loop above would cost four
        // instructions more per logit, a second run of that loop eight registers and with them a wave per SIMD.  With every
        // key that far down, 32 x 2781 x 64 bf16 takes 574 us instead of 60, less than the 786 us of scores on the vector ALU.)
        const uint64_t few = __ballot(mine && sum < (float)group * (float)L * 0x1p-102f);      // alike in all four waves
        if (__builtin_expect(few != 0, 0)) {
            __syncthreads();                         // fold_a has been read
            for (uint64_t todo = few; todo != 0;) {
                int r[FEW], key[FEW];
#pragma unroll
                for (int n = 0; n < FEW; ++n) {      // fewer left: the last one again
                    r[n] = (n == 0 || todo != 0) ? __builtin_ctzll(todo) : r[n > 0 ? n - 1 : 0];
                    key[n] = s0 + r[n];
                    todo &= todo - 1;
                }
                float f[FEW] = {};
                for (int g = 0; g < group; ++g) {
                    const size_t row0 = ((size_t)h * group + g) * L;
                    weights_of_keys(q + row0 * d, k + (size_t)h * L * d, lse2 + row0, key, R0, L, d, scale2, lse_scale, f);
                }
#pragma unroll
                for (int n = 0; n < FEW; ++n) {
#pragma unroll
                    for (int off = 1; off < 64; off <<= 1) f[n] += __shfl_xor(f[n], off);
                    if (lane == 0) fold_a[wave][r[n]] = f[n];
                }
            }
            __syncthreads();
            if ((few >> lane) & 1) sum = fold();
        }
        if (wave != 0 || !mine) return;
    }
    out[(size_t)h * L + s0 + lane] = sum;
}

}  // namespace lookm

namespace lookm_host {

int launch_scores_mfma(const void* q, const void* k, int H, int kv_heads, int L, int d, int R0, float* lse,
                       const float* lse_in, float* scores, float* rnorm, float* scratch, size_t scratch_floats,
                       const uint8_t* mask, int M, int32_t* lists, ScoreParts* parts, hipStream_t st);
size_t scores_mfma_scratch_floats(int H, int L, bool least);

// The kernel of a pass for these strips, each of up to `streamed` rows.  Remainders of fp32 parts come from the dot instruction: fewer
// instructions, a longer chain.  At 40 to 64 dims that is a loss where long strips keep three and four waves a SIMD busy.  By strips per
// compute unit, subtracted / dots, us: 3 heads x 5308 x 64 (1.9) pass 1 54.9 / 52.3, pass 2 57.0 / 55.0; 4 (2.6) 58.7 / 60.8, 59.2 / 61.2; 3 x
// 9916 x 48 (3.6) 119 / 126, 120 / 123; 8 x 5308 x 64 (5.2) 96.8 / 98.5, 94.8 / 93.5; 24 query heads on 6 x 3576 x 64 pass 1 (10.5) 131 /
// 137, pass 2 (2.6) 153 / 159; 40 on 10 x 3384 pass 2 (4.1), layer, 306 / 315; 24 x 5308 x 64 (15.6) 271 / 268, 269 / 266.  Short strips, whole layers: 4 heads x 4156 x 64 (2.0) 126 / 123, 32 x
// 956 (3.8) 66.0 / 64.8, 64 x 1692 (13) 219 / 215.  (x 32: dots gain 2 to 6 % throughout, x 128 3 to 4 %.)
template <int PASS, typename T, int KS, int CG>
static auto score_kernel(long strips, long streamed)
{
    if constexpr (sizeof(T) == 4 && (KS == 3 || KS == 4) && CG == 2)
        if (streamed >= 3500 && strips > 576 && strips <= (PASS == 1 ? 2816 : 1152)) return &lookm::k_score_any<PASS + lookm::SUBTRACT, T, KS, CG>;
    return &lookm::k_score_any<PASS, T, KS, CG>;
}

template <typename T>
static int launch_scores_any(const T* q, const T* k, int H, int kv_heads, int L, int d, int R0, float* lse,
                             const float* lse_in, float* scores, float* rnorm, hipStream_t st)
{
    const LaunchCheck check;
    const int group = H / kv_heads;
    const float scale2 = lookm::kLog2e / sqrtf((float)d);
    const size_t norm_rows = rnorm ? (size_t)kv_heads * L : 0, norm_blocks = (norm_rows + 31) / 32;   // they ride with the first launch
    auto units = [](int heads, int strips) { return (unsigned)((heads >= 8 ? (heads + 7) / 8 * 8 : heads) * strips); };
    const int together = (int)std::min<size_t>(64, std::max<size_t>(1, (size_t)(2 << 20) / ((size_t)L * d * sizeof(T))));
    auto strips = [&](int rows) { return (long)((L - R0 + rows - 1) / rows) * H; };
    lookm::with_frag_shape<T>(d, strips, [&](auto steps, auto groups) {
        constexpr int KS = decltype(steps)::value, CG = decltype(groups)::value;
        const int nS = (L + 16 * CG - 1) / (16 * CG);
        if (!lse_in) {
            const int n1 = nS - R0 / (16 * CG);       // strips with a query row that counts (observation window)
            hipLaunchKernelGGL((score_kernel<1, T, KS, CG>((long)H * n1, L)), wide_grid(units(H, n1) + norm_blocks), dim3(256), 0, st, q, k, H, group,
                               L, R0, d, scale2, (const float*)nullptr, 1.0f, lse, n1, together, units(H, n1), norm_rows, rnorm);
            mark(LOOKM_K_SCORE_LSE);
        }
        // a caller-supplied row log-sum-exp is natural-log: one factor log2(e) brings it to the kernels' base
        hipLaunchKernelGGL((score_kernel<2, T, KS, CG>((long)kv_heads * nS, (long)group * (L - R0))), wide_grid(units(kv_heads, nS) + (lse_in ? norm_blocks : 0)), dim3(256), 0,
                           st, q, k, kv_heads, group, L, R0, d, scale2, lse_in ? lse_in : lse, lse_in ? lookm::kLog2e : 1.0f,
                           scores, nS, together, units(kv_heads, nS), lse_in ? norm_rows : 0, rnorm);
        mark(LOOKM_K_SCORE_COLSUM);
    });
    return check.status();
}

size_t scores_scratch_floats(int H, int L, int d, lookm_dtype dt, bool least)
{
    return (dt == LOOKM_BF16 && d == 128) ? scores_mfma_scratch_floats(H, L, least) : 0;
}

int launch_scores(const void* q, const void* k, int H, int kv_heads, int L, int d, lookm_dtype dt, int first_row,
                  float* lse, const float* lse_in, float* scores, float* rnorm, float* scratch, size_t scratch_floats,
                  const uint8_t* mask, int M, int32_t* lists, ScoreParts* parts, hipStream_t st)
{
    const int R0 = first_row;
    if (dt == LOOKM_BF16) {
        if (d == 128)
            return launch_scores_mfma(q, k, H, kv_heads, L, d, R0, lse, lse_in, scores, rnorm, scratch, scratch_floats, mask, M, lists, parts, st);
        return launch_scores_any((const lookm::bf16_t*)q, (const lookm::bf16_t*)k, H, kv_heads, L, d, R0, lse, lse_in, scores,
                                 rnorm, st);
    }
    return launch_scores_any((const float*)q, (const float*)k, H, kv_heads, L, d, R0, lse, lse_in, scores, rnorm, st);
}

}  // namespace lookm_host
