// Accumulated attention scores (Section 3.2, Eq. 4) on the gfx950 matrix cores: bf16, head_dim 128.
//
// Both passes are the same machine with the roles of Q and K swapped.  A workgroup (4 waves)
// owns 256 "stationary" rows - query rows in pass 1, key rows in pass 2 - whose MFMA B-operand
// fragments stay in registers (64 rows x 128 dims per wave = 64 VGPRs), and streams the other
// tensor past them in 64-row tiles through double-buffered LDS as the A operand.  The MFMA is
// v_mfma_f32_16x16x32_bf16: a 32-row block of the streamed tensor against the wave's 64 stationary rows is
// eight 16x16 tiles (two groups of 16 streamed rows x four groups of 16 stationary rows), and of every tile a
// lane (c = lane % 16, q = lane / 16) holds the streamed rows 4q .. 4q+3 against stationary row c.  A lane's
// 32 accumulator values of a block thus belong to FOUR stationary rows, eight streamed rows each, and both
// reductions of the method stay in-lane:
//   pass 1: running (max, sum) of 2^(c q.k) over the keys of a query row   -> lse2[i]
//   pass 2: running sum of 2^(c q.k - lse2[i]) over the query rows of a key -> A_s[j]
// The four lanes that share a stationary row (equal c) are combined once, after the loop.  (The 32x32x16 form
// of the instruction, with which a lane holds 16 streamed rows of two stationary rows, does the same work in
// the same registers, but this chip sustains 13 % less of it under this load, measured with random operands;
// with the epilogues the two score passes together are 6 % faster this way.)
// Nothing is atomically accumulated; every sum has a fixed order, so results are bitwise
// repeatable.  c = log2(e)/sqrt(d) folds the softmax scale into the exp2 argument.
#include "score_parts.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace lookm {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

static_assert(BX == 64, "the lse staging of pass 2 is done by wave 0, one row per lane");
constexpr int XROW = 128;       // LDS row = 256 B, unpadded; the 16-byte chunk c of row r sits at chunk c ^ (r & 7),
                               // so 16-byte reads of 8 consecutive rows at the same c hit all 32 banks once

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// Epilogues of a finished block: acc[rg][cg], rg = which 16 of the block's 32 streamed rows, cg = which 16 of the
// wave's 64 stationary rows.  Entry i of acc[rg][cg] is streamed row xq + 16*rg + i (xq = block start + 4q) against
// this lane's stationary row of group cg, whose position is sP[cg].

// A block on the diagonal: logits outside the causal region become -inf (weight 0), in place and ahead of the one epilogue
// that every block runs - with an epilogue of its own for masked blocks the running values met on two paths, a register
// copy for each of them in every block.
template <int PASS>
__device__ __forceinline__ void mask_block(f32x4 (&acc)[2][4], int xq, const int (&sP)[4])
{
#pragma unroll
    for (int cg = 0; cg < 4; ++cg)
#pragma unroll
        for (int rg = 0; rg < 2; ++rg)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int x = xq + 16 * rg + i;
                if (PASS == 1 ? x > sP[cg] : x < sP[cg]) acc[rg][cg][i] = -INFINITY;
            }
}

//   PASS 2: running sums of 2^(c*(s - b_i)) over the query rows of the lane's four keys, b_i = lse2_i / c; the
//           accumulators arrive with -b_i already in them (the MFMA chain starts from it instead of from zero),
//           so no per-row value has to be held in registers here.
__device__ __forceinline__ void colsum_block_epilogue(const f32x4 (&acc)[2][4], float scale2, float (&run)[4])
{
#pragma unroll
    for (int cg = 0; cg < 4; ++cg) {
        float sum;   // (started from its first term: 0 + x is an addition the compiler may not drop)
#pragma unroll
        for (int rg = 0; rg < 2; ++rg)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float p = __builtin_amdgcn_exp2f(acc[rg][cg][i] * scale2);
                sum = (rg == 0 && i == 0) ? p : sum + p;
            }
        run[cg] += sum;
    }
#pragma unroll
    for (int cg = 0; cg < 4; ++cg) asm volatile("" : "+v"(run[cg]));   // here, not sunk behind the next block's MFMAs
}

// Pass 1, a finished block (32 streamed keys against the lane's four query rows).
// The reference of a running sum is refreshed lazily: a block is first summed against the row's current reference m;
// only if a sum overflows (the first block of a row, where m is still "minus infinity", or a logit more than 64
// binades above the reference) is the block maximum taken and the running sum rescaled.  The result is the same up
// to rounding - a float sum keeps its relative precision at any magnitude below 2^64 - and the common case saves
// the maximum over the block.  One wave-uniform test covers the whole block (a branch on a vector result drains the
// wave's vector pipeline); the refresh is valid for a row that did not overflow as well.  A NaN needs no refresh: it
// reaches the running sum either way.
__device__ __forceinline__ void lse_refresh(const f32x4& lo, const f32x4& hi, float scale2, float& m, float& l, float& sum)
{
    const float bm = fmaxf(fmaxf(fmaxf(fmaxf(lo[0], lo[1]), lo[2]), fmaxf(fmaxf(lo[3], hi[0]), hi[1])), fmaxf(hi[2], hi[3]));
    const float mn = fmaxf(m, bm * scale2);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) s += __builtin_amdgcn_exp2f(fmaf(lo[i], scale2, -mn));
#pragma unroll
    for (int i = 0; i < 4; ++i) s += __builtin_amdgcn_exp2f(fmaf(hi[i], scale2, -mn));
    l = fmaf(l, __builtin_amdgcn_exp2f(m - mn), s);
    m = mn;
    sum = 0.f;                 // in l already, with one rounding
}

__device__ __forceinline__ void lse_block_epilogue(const f32x4 (&acc)[2][4], float scale2, float (&m)[4], float (&l)[4])
{
    float sum[4];
#pragma unroll
    for (int cg = 0; cg < 4; ++cg) {
#pragma unroll
        for (int rg = 0; rg < 2; ++rg)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float p = __builtin_amdgcn_exp2f(fmaf(acc[rg][cg][i], scale2, -m[cg]));
                sum[cg] = (rg == 0 && i == 0) ? p : sum[cg] + p;   // (0 + x is an addition the compiler may not drop)
            }
    }
    const float top = fmaxf(fmaxf(fmaxf(sum[0], sum[1]), sum[2]), sum[3]);
    if (__builtin_expect(__any(top > 1.8e19f), 0)) {     // wave-uniform
#pragma unroll
        for (int cg = 0; cg < 4; ++cg) lse_refresh(acc[0][cg], acc[1][cg], scale2, m[cg], l[cg], sum[cg]);
    }
#pragma unroll
    for (int cg = 0; cg < 4; ++cg) l[cg] += sum[cg];
}

// ---- work decomposition -------------------------------------------------------------------------------
// A strip is 256 stationary rows; its streamed range (keys 0..strip end in pass 1, query rows strip
// start..L in pass 2) is 4..L/64 tiles long.  The streamed axis is cut at multiples of CT = C*64 rows
// into chunks, one workgroup per (strip, chunk), so that no workgroup is much longer than the average
// (the longest strip alone would otherwise set the kernel's duration).  Chunk boundaries are the same
// for every strip, and work is enumerated chunk-major, so the workgroups resident on an XCD at one
// time stream the SAME rows of the same head and share them in that XCD's L2.  Each workgroup writes a
// partial result per stationary row; a small second kernel folds a strip's chunks together in order.
//
// With an observation window only the query rows R0 .. L-1 count (R0 = 0: all rows, Eq. 4 as printed): pass 1
// then needs only the strips that hold such rows, and pass 2 streams a strip's query rows from max(strip start,
// R0) on, so the chunks below R0 are empty for every strip.
__host__ __device__ inline int first_chunk(int pass, int t, int CT, int R0)
{
    return (pass == 1) ? 0 : max(t * BS, R0) / CT;
}
__host__ __device__ inline int strip_chunks(int pass, int t, int L, int CT, int R0)
{
    if (pass == 1) return ((t + 1) * BS > R0) ? (min(L, (t + 1) * BS) + CT - 1) / CT : 0;
    return (L + CT - 1) / CT - max(t * BS, R0) / CT;
}

// The matrix pipe and the vector ALU of a SIMD overlap ACROSS waves far better than within one (measured), so a
// wave's arithmetic stays in two phases - MFMA chains, then the epilogue - and the kernel is sized for three
// resident waves per SIMD; what a wave does overlap with its own arithmetic is memory latency (LDS fragment
// fetches one block ahead, tile loads one tile ahead).
//   PASS 1 writes part_a = running max, part_b = running sum (base-2 domain) per (chunk, stationary row).
//   PASS 2 writes part_a = partial column sum per (chunk, stationary row).  Its stationary rows are keys: when
//   `rnorm` is given, the workgroup of a strip's first chunk also writes rnorm[h, j] = 1 / ||k_j|| (0 for a
//   zero key) for the matching of Eq. 9, from the registers it holds anyway - the keys are not read again for it.
// ---- scores for the competing keys only -------------------------------------------------------------------
// Selection ranks only the image tokens before the recent window (Eq. 5-8: text tokens and the window are
// conserved whatever their score).  When the caller does not ask for the scores themselves, pass 2 therefore
// runs over those keys alone: its strips are 256 consecutive entries of the ascending list of competing positions
// instead of 256 consecutive positions, and everything else - chunk boundaries, the tiles a key's column sum runs
// over, the order of every addition - is unchanged, so the scores of the competing keys come out bit for bit as
// on the dense path.  The lists are built from the modality mask by one extra workgroup of pass 1 (or by a small
// kernel of its own when pass 1 is skipped):
//   lists[0] = number of competing keys, lists[1] = number of protected keys,
//   lists[LIST_HEAD .. +L) competing positions ascending, lists[LIST_HEAD + L .. +L) protected positions ascending.

// By a workgroup of NT threads.  A wave classifies 64 consecutive positions at a time (coalesced mask bytes, one ballot),
// eight such rows in flight; the ballots stay in LDS, their counts are scanned, and a second sweep writes both lists.
// (With a contiguous range of positions per thread instead, 12644 positions took a kernel of its own 12.7 us, now 6.2 us.)
constexpr int LIST_WORDS = LOOKM_MAX_L / 64;
template <int NT>
__device__ __forceinline__ void build_key_lists(const uint8_t* __restrict__ mask, int L, int M, int32_t* __restrict__ lists,
                                                uint64_t* words /* LDS, LIST_WORDS */, int* before /* LDS, LIST_WORDS + NT / 64 */)
{
    constexpr int NW = NT / 64, PER = (LIST_WORDS + NT - 1) / NT;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, n = (L + 63) / 64;
    int* wsum = before + LIST_WORDS;
    for (int j0 = wave; j0 < n; j0 += NW * 8) {
        uint8_t b[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) b[u] = mask[min((j0 + NW * u) * 64 + lane, L - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int j = j0 + NW * u;
            const uint64_t w = __ballot(b[u] != 0 && j * 64 + lane < L - M);      // image tokens before the window
            if (lane == 0 && j < n) words[j] = w;
        }
    }
    __syncthreads();
    int count[PER], incl = 0;                                // thread t looks after the words t * PER ..
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int j = tid * PER + u;
        count[u] = (j < n) ? __popcll(words[j]) : 0;
        incl += count[u];
    }
    int own = incl;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int run = incl - own, all = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        run += (w < wave) ? wsum[w] : 0;
        all += wsum[w];
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (tid * PER + u < LIST_WORDS) before[tid * PER + u] = run;
        run += count[u];
    }
    if (tid == 0) { lists[0] = all; lists[1] = L - all; }
    __syncthreads();
    for (int j = wave; j < n; j += NW) {
        const uint64_t w = words[j];
        const int pos = j * 64 + lane, c = before[j] + mask_rank(w);
        if ((w >> lane) & 1ull) lists[LIST_HEAD + c] = pos;
        else if (pos < L) lists[LIST_HEAD + L + pos - c] = pos;
    }
}

__global__ void __launch_bounds__(1024) k_score_lists(const uint8_t* __restrict__ mask, int L, int M, int32_t* __restrict__ lists)
{
    __shared__ uint64_t words[LIST_WORDS];
    __shared__ int before[LIST_WORDS + 16];
    build_key_lists<1024>(mask, L, M, lists, words, before);
}

template <int PASS, bool SPARSE>
__global__ void __launch_bounds__(256, 3)
k_score_mfma(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, int H, int group, int L, int R0, float scale2,
             int C, int U, const float* __restrict__ lse2, float lse_scale, float* __restrict__ part_a,
             float* __restrict__ part_b, float* __restrict__ rnorm, const uint8_t* __restrict__ modality, int M,
             int32_t* __restrict__ lists)
{
    // Two tiles as separate arrays, with the buffer of a tile known at compile time (the tile loop is unrolled by
    // two): the compiler then sees that a fragment read of one array cannot alias the loads in flight to the
    // other.  With one array indexed by a run-time buffer number it waits for every outstanding load before a
    // tile's first LDS read, which serialises the prefetch with the MFMA block of the same wave.
    __shared__ __attribute__((aligned(16))) bf16_t xs0[BX * XROW];
    __shared__ __attribute__((aligned(16))) bf16_t xs1[BX * XROW];
    __shared__ __attribute__((aligned(16))) float xl0[BX];   // pass 2: -lse2[i] of the streamed query rows
    __shared__ __attribute__((aligned(16))) float xl1[BX];
    __shared__ __attribute__((aligned(16))) bf16_t turn[4][16 * XROW];   // stationary rows changing lanes
    __shared__ int spos[SPARSE ? 4 * 256 : 1];   // sparse pass 2: positions of every lane's four stationary rows

    // pass 1 with a mask: the launch has one workgroup more, which builds the key lists for pass 2
    if (PASS == 1 && modality != nullptr && blockIdx.x == gridDim.x - 1) {
        build_key_lists<256>(modality, L, M, lists, reinterpret_cast<uint64_t*>(xs0), reinterpret_cast<int*>(xs1));
        return;
    }
    // pass 2 with lists: stationary rows are entries of the list of competing positions
    static_assert(PASS == 2 || !SPARSE, "only pass 2 has a sparse form");
    constexpr bool sparse = SPARSE;
    const int NC = sparse ? lists[0] : L;                 // stationary rows in all
    const int32_t* clist = lists + LIST_HEAD;

    // Consecutive workgroup ids go to consecutive XCDs.  With 8 or more heads, XCD x works through heads
    // x, x+8, ... one at a time, so its L2 holds one head's current chunk; with fewer heads each head
    // gets 8/H XCDs that share its units round-robin.
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    int h, e;
    if (H >= 8) {
        h = (j / U) * 8 + xcd;
        e = j % U;
    } else {
        const int xph = 8 / H;            // XCDs per head
        h = xcd / xph;
        e = j * xph + xcd % xph;
    }
    if (h >= H || e >= U) return;
    const int nS = (L + BS - 1) / BS, CT = C * BX;
    int g = (PASS == 1) ? 0 : R0 / CT, tile = 0;
    for (;; ++g) {      // chunk-major enumeration: all strips that touch chunk g, then chunk g+1, ...
        const int t_first = (PASS == 1) ? max((g * CT) / BS, R0 / BS) : 0;
        const int cnt = (PASS == 1) ? nS - t_first : min(nS, ((g + 1) * CT + BS - 1) / BS);
        if (e < cnt) { tile = t_first + e; break; }
        e -= cnt;
    }
    const int s0 = tile * BS;
    const int n_chunks_total = (L + CT - 1) / CT;
    // slot of this (chunk, strip) in the partial arrays [h][chunk][strip][256]; pass 1 under an observation window
    // only has the strips from the window's first one on, and indexes them from there
    const int t_base = (PASS == 1) ? R0 / BS : 0, nSp = nS - t_base;
    const int u = g * nSp + (tile - t_base);
    // h runs over the query heads; with grouped query heads, `group` consecutive ones read key head h / group
    const bf16_t* qh = q + (size_t)h * L * SD;
    const bf16_t* kh = k + (size_t)(h / group) * L * SD;
    const bf16_t* S = (PASS == 1) ? qh : kh;   // stationary tensor
    const bf16_t* X = (PASS == 1) ? kh : qh;   // streamed tensor
    const float* lse_h = lse2 + (size_t)h * L;

    // the wave number is uniform across a wave: taken through a scalar register, everything derived from it (the
    // wave's first row, loop bounds, LDS addresses) stays in scalar registers and scalar branches
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, q4 = lane >> 4,
              c16 = lane & 15;   // this lane: column c16 of every 16x16 tile, rows 4*q4 .. 4*q4+3
    const int w0 = s0 + wave * 64;

    // The strip's first row decides where its streamed range starts (sparse: a list entry).
    const int p_strip = !sparse ? s0 : (s0 < NC) ? __builtin_amdgcn_readfirstlane(clist[min(s0, L - 1)]) : 0;
    const int strip_begin = (PASS == 1) ? 0 : (p_strip / BX) * BX;
    const int strip_end = (PASS == 1) ? min(L, s0 + BS) : L;
    const int x_begin = max(max(strip_begin, g * CT), (PASS == 2) ? (R0 / BX) * BX : 0);   // tile-aligned
    const int x_end = min(strip_end, (g + 1) * CT);
    // (sparse) no such strip of competing keys, or the chunk ends before the strip's first key: such a unit runs no
    // tile and writes partials that nothing reads (an early exit here costs the kernel its register budget)
    const bool idle = sparse && (s0 >= NC || x_end <= x_begin);

    // Positions of this lane's four stationary rows (row 16*cg + c16 of the wave, cg = 0..3) and of the wave's first
    // and last row: row numbers themselves on the dense path, list entries on the sparse one (rows past the end of the
    // list: a position past the prompt, which no query row reaches).
    int p_wave_lo = w0, p_wave_hi = w0 + 63;
    if (sparse) {
        // wave-uniform values: kept in scalar registers
        p_wave_lo = (w0 < NC) ? __builtin_amdgcn_readfirstlane(clist[min(w0, NC - 1)]) : 0x3fffffff;
        p_wave_hi = (w0 < NC) ? __builtin_amdgcn_readfirstlane(clist[min(w0 + 63, NC - 1)]) : 0x3fffffff;
    }
    // the position of stationary row cg of this lane (sparse: from LDS, see below)
    auto stationary_pos = [&](int cg) { return sparse ? spos[cg * 256 + tid] : w0 + 16 * cg + c16; };

    // stationary fragments: of row 16*cg + c16, the dims 32*ks + 8*q4 .. +7 (the B operand of MFMA step ks).  The rows are
    // loaded sixteen lanes to a row and change lanes through LDS (4 KB per wave, no barrier): loads in fragment order, sixteen
    // rows per instruction, run at 15.5 B per clock and compute unit, a workgroup's 64 KB at 1.8 us, these at 54 B, 0.5 us -
    // of the L1 time that the tiles of the other workgroups need too.
    if (sparse)
#pragma unroll
        for (int cg = 0; cg < 4; ++cg) {
            // the per-lane positions are only needed again where a tile touches the diagonal (and for the norms):
            // parked in LDS meanwhile (each lane reads back what it wrote itself, so no barrier is involved)
            const int row = w0 + 16 * cg + c16;
            spos[cg * 256 + tid] = (row < NC) ? clist[row] : 0x3fffffff;
        }
    bf16x8 sf[4][4];
    {
        // Pass 1: a wave wholly past the end has zeros - a buffer of no bytes, which needs no memory.  (Under an observation
        // window the last strip is all there is: a window of 64 in 12644 tokens, where two waves of four lie past the end,
        // 40.1 -> 38.2 us.)
        const auto srsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(S), 0, (PASS == 1 && w0 >= L) ? 0 : L * (SD * 2), 0x00020000);
        u32x4 rows[4][4];
        auto load_rows = [&](auto&& offset) {     // offset(r): scalar and per-lane byte offset of row r (+ q4) of the wave
#pragma unroll
            for (int cg = 0; cg < 4; ++cg)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int2 o = offset(16 * cg + 4 * i);
                    rows[cg][i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(srsrc, o.y, o.x, 0));
                }
        };
        if (sparse)                               // rows past the end of the list repeat its last one: nothing reads their results
            load_rows([&](int r) { return make_int2(0, (int)min((unsigned)clist[min(w0 + r + q4, max(NC, 1) - 1)], (unsigned)(L - 1)) * (SD * 2) + c16 * 16); });
        else if (s0 + BS <= L)                    // a whole strip: no arithmetic per row
            load_rows([&](int r) { return make_int2((w0 + r) * (SD * 2), lane * 16); });
        else                                      // rows past the end repeat the last one
            load_rows([&](int r) { return make_int2(0, min(w0 + r + q4, L - 1) * (SD * 2) + c16 * 16); });
        bf16_t* mine = turn[wave];
        const bf16_t* theirs = mine + unknown_zero();
#pragma unroll
        for (int cg = 0; cg < 4; ++cg) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<u32x4*>(&mine[(4 * i + q4) * XROW + (c16 ^ ((4 * i + q4) & 7)) * 8]) = rows[cg][i];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                sf[cg][ks] = as_bf16x8(*reinterpret_cast<const uint4*>(&theirs[c16 * XROW + ((4 * ks + q4) ^ (c16 & 7)) * 8]));
        }
    }

    const int n_it = idle ? 0 : (x_end - x_begin + BX - 1) / BX;

    // Staging goes from global memory straight into LDS (buffer_load_dwordx4 lds): the 64 lanes of a wave
    // fill 1 KB = 4 consecutive LDS rows, lane l landing at chunk l%16 of row l/16, so the swizzle is applied
    // on the global side: the lane fetches chunk (l%16) ^ (row & 7) of its row.  Rows past the end re-read the
    // last row (their contribution is masked out or weighted by 2^-inf).  No staging registers, no LDS stores, and with
    // a buffer descriptor no address arithmetic: a lane's offset inside a tile never changes, the rest is scalar.
    // (32 heads x 12644, with one epilogue per block instead of a masked and a plain one, and in pass 2 the blocks written
    // out instead of a loop over the two, in which a fragment read waited for the loads of the next tile: pass 1
    // 599 -> 591 us, pass 2 530 -> 513 us, bit-identical; pass 2's vector instructions per block 119 -> 108.)
    constexpr int NLD = BX / 16;   // 1 KB pieces per wave and tile
    float stage_l = 0.f;
    // byte offset of this lane's 16 bytes inside a tile: row (wave*4 + lane/16) of the first 1 KB piece, swizzled chunk
    // (the 16 rows between two pieces do not change row & 7)
    // The lane number afresh (two instructions), where values derived from it are needed once in a while: no register has
    // to hold them meanwhile.  With the registers all taken the compiler otherwise parks them in scratch memory, and every
    // reload waits for the tile loads in flight.
    auto lane_again = [&]() {
        int t = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        asm volatile("" : "+v"(t));
        return t;
    };
    const auto xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(X), 0, L * (SD * 2), 0x00020000);
    auto lane_offset = [&](int t) {
        const int row = wave * 4 + (t >> 4);
        return row * (SD * 2) + ((t & 15) ^ (row & 7)) * 16;
    };
    const int lane_off = lane_offset(lane);
    auto load_tile = [&](int x0, bf16_t* xsb) {
        if (x0 + BX <= L) {          // scalar test: a whole tile inside the tensor needs no clamping
            const int o = (PASS == 1) ? lane_offset(lane_again()) : lane_off;
#pragma unroll
            for (int i = 0; i < NLD; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    xrsrc, (__attribute__((address_space(3))) void*)&xsb[(i * 4 + wave) * 4 * XROW], 16, o,
                    x0 * (SD * 2) + i * 16 * SD * 2, 0, 0);
        } else {                     // the tensor's last tile: rows past the end re-read the last row
            const int o = lane_offset(lane_again()), row = o >> 8, chunk = o & 255;   // SD * 2 = 256 bytes per row
#pragma unroll
            for (int i = 0; i < NLD; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    xrsrc, (__attribute__((address_space(3))) void*)&xsb[(i * 4 + wave) * 4 * XROW], 16,
                    min(x0 + i * 16 + row, L - 1) * (SD * 2) + chunk, 0, 0, 0);
        }
        // Pass 2 also needs lse2 of the tile's rows: wave 0 (threads 0 .. BX-1, a scalar test) loads one value per
        // lane here, unconditionally (rows outside the tensor read its last row), and store_tile puts it into LDS at
        // the end of the previous tile.  Nothing may touch the loaded value before that: a use right after the load
        // would make the wave wait for everything it has just issued, the tile's rows included - hence the empty asm
        // in store_tile, which keeps the compiler from moving the arithmetic up here.
        if (PASS == 2 && wave == 0) stage_l = lse_h[min(x0 + lane_again(), L - 1)];
    };
    // x0: first row of the tile that was loaded.  Value stored: -lse2_i / c (the start of the MFMA chains of pass 2);
    // rows outside [R0, L) get -inf and contribute nothing.
    auto store_tile = [&](float* xlb, int x0) {
        if (PASS == 2 && wave == 0) {
            float v = stage_l;
            asm volatile("" : "+v"(v));
            const int t = lane_again();
            xlb[t] = (x0 + t < L && x0 + t >= R0) ? -v * lse_scale : -INFINITY;
        }
    };

    float m[4] = {-1e30f, -1e30f, -1e30f, -1e30f}, l[4] = {0.f, 0.f, 0.f, 0.f};   // pass 1 state per stationary row of this lane
    float run[4] = {0.f, 0.f, 0.f, 0.f};                                            // pass 2 state

    load_tile(x_begin, xs0);
    store_tile(xl0, x_begin);
    if (PASS == 2 && rnorm != nullptr && g == max(strip_begin, (R0 / BX) * BX) / CT && h % group == 0) {
        // A key row's 128 dims sit in the four lanes of equal c16: lane q4 holds the 8-dim groups q4, 4 + q4, 8 + q4
        // and 12 + q4.  The sum of squares is taken in the order of the stand-alone norm kernel (k_rnorm: eight
        // partial sums, number p over the groups p and p + 8, then a pairwise tree), so both give the same bits
        // and the stage call lookm_nearest reproduces the matching of the whole path exactly.
#pragma unroll
        for (int cg = 0; cg < 4; ++cg) {
            double part[2];   // partial sums number q4 and 4 + q4, in binary64 as in k_rnorm
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                double ss = 0.0;
#pragma unroll
                for (int rep = 0; rep < 2; ++rep) {      // group 4*j + q4 (step j), then group 8 + 4*j + q4 (step j + 2)
                    const uint4 v = __builtin_bit_cast(uint4, sf[cg][j + 2 * rep]);
                    const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float lo = __uint_as_float(w4[i] << 16), hi = __uint_as_float(w4[i] & 0xffff0000u);
                        ss = fma((double)lo, (double)lo, ss);
                        ss = fma((double)hi, (double)hi, ss);
                    }
                }
                part[j] = ss;
            }
            // (p0 + p1) + (p2 + p3) and (p4 + p5) + (p6 + p7), then their sum
            double lo4 = part[0] + __shfl_xor(part[0], 16), hi4 = part[1] + __shfl_xor(part[1], 16);
            lo4 += __shfl_xor(lo4, 32);
            hi4 += __shfl_xor(hi4, 32);
            const double ss = lo4 + hi4;
            const int row = stationary_pos(cg);
            if (q4 == 0 && row < L) rnorm[(size_t)(h / group) * L + row] = inverse_norm(ss);
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the direct-to-LDS loads have landed
    __syncthreads();

    // element offsets of this lane's first two fragments inside its LDS row (swizzled chunks 4*ks + q4); the
    // chunks of steps 2 and 3 lie 8 chunks after those of steps 0 and 1
    int frag_off[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) frag_off[ks] = ((4 * ks + q4) ^ (c16 & 7)) * 8;

    // Which tiles need the mask (wave-uniform, so the choice is a scalar branch):
    //   pass 1, keys stream upwards: tiles with x0 + BX - 1 <= w0 hold only keys at or before every query row of
    //   this wave, the tiles after them touch the diagonal;
    //   pass 2, query rows stream upwards from the diagonal: tiles with x0 >= w0 + 63 need no mask.
    int plain_from, plain_to;
    if (PASS == 1) {
        const int n_plain = (w0 - x_begin + 1) / BX;        // largest count with x_begin + BX*count - 1 <= w0
        plain_from = 0;
        plain_to = max(0, min(n_plain, n_it));
    } else {
        const int n_masked = (min(p_wave_hi, L) - x_begin + BX - 1) / BX;
        plain_from = max(0, min(n_masked, n_it));
        plain_to = n_it;
    }
    // fragments of one block of 32 streamed rows (the A operands of its 32 MFMAs: row 16*rg + c16 of the block,
    // dims 32*ks + 8*q4 .. +7), fetched one block ahead
    bf16x8 a[2][4];
    auto fetch_group = [&](const bf16_t* tile_rows, int rb, int rg) {
        const bf16_t* ap = &tile_rows[(rb * 32 + 16 * rg + c16) * XROW];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            a[rg][ks] = as_bf16x8(*reinterpret_cast<const uint4*>(ap + frag_off[ks]));
            a[rg][ks + 2] = as_bf16x8(*reinterpret_cast<const uint4*>(ap + frag_off[ks] + 64));
        }
    };
    auto fetch = [&](const bf16_t* tile_rows, int rb) {
        fetch_group(tile_rows, rb, 0);
        fetch_group(tile_rows, rb, 1);
    };
    // pass 2: what the MFMA chains of a block start from, -lse2_i / c of the lane's streamed rows, fetched with the fragments
    f32x4 init[2];
    auto fetch_init = [&](const float* tile_l, int rb) {
#pragma unroll
        for (int rg = 0; rg < 2; ++rg)
            init[rg] = __builtin_bit_cast(f32x4, *reinterpret_cast<const float4*>(&tile_l[rb * 32 + 16 * rg + 4 * q4]));
    };
    if (n_it > 0) {
        fetch(xs0, 0);
        if (PASS == 2) fetch_init(xl0, 0);
    }

    // One tile, with its LDS buffer known at compile time.  Tiles that touch the diagonal evaluate the causal
    // condition per element in their epilogues; tiles known to lie entirely inside the causal region run the same
    // epilogue minus the comparisons.  The choice is wave-uniform and made by a scalar branch around the epilogue
    // only, so that there is one tile body per buffer (with a body per mask variant the fragments carried from one
    // tile to the next would have to meet in the same registers on four paths, and the kernel no longer fits).
    auto tile_step = [&](auto buf_tag, int it) {
        constexpr int BUF = decltype(buf_tag)::value;
        bf16_t* cur = BUF ? xs1 : xs0;
        bf16_t* nxt = BUF ? xs0 : xs1;
        float* cur_l = BUF ? xl1 : xl0;
        float* nxt_l = BUF ? xl0 : xl1;
        const int x0 = x_begin + it * BX;
        if (it + 1 < n_it) load_tile(x0 + BX, nxt);
        // wave-uniform: a tile that lies entirely outside the causal region is not computed at all
        const bool mask = !(it >= plain_from && it < plain_to);
        const bool skip = mask && ((PASS == 1) ? (x0 > w0 + 63) : (x0 + BX - 1 < p_wave_lo));

        // End of the tile's LDS reads: wait for the next tile's loads, meet the other waves, and fetch the next
        // tile's first fragments - before the epilogue of this tile's second block, which hides their latency.
        auto finish_tile = [&]() {
            if (it + 1 < n_it) store_tile(nxt_l, x0 + BX);
            __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the next tile's direct-to-LDS loads have landed
            __syncthreads();
            // unconditional: after the last tile this reads an old tile and the values are never used
            fetch(nxt, 0);
            if (PASS == 2) fetch_init(nxt_l, 0);
        };
        if (!skip) {
            // Two blocks of 32 streamed rows; the fragments of block 0 are in `a` already (fetched by the previous
            // tile, or before the loop).  A block's fragments are dead once its MFMAs have been issued, so the next
            // block's are fetched into the same registers right away and their LDS latency passes under the
            // epilogue.  The scheduling barriers keep the compiler from undoing the order, and from holding more
            // than one block's values at a time: the kernel has to stay within 168 VGPRs.
            f32x4 acc[2][4];
            // the MFMA chains of a block start from zero in pass 1 and from -lse2_i / c of the lane's streamed rows in pass 2;
            // step by step over all eight tiles, so that a tile's next MFMA is eight instructions away
            auto multiply = [&]() {
                const f32x4 zero = {0.f, 0.f, 0.f, 0.f};   // an inline constant of the instruction, no registers
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int cg = 0; cg < 4; ++cg)
#pragma unroll
                        for (int rg = 0; rg < 2; ++rg)
                            acc[rg][cg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                a[rg][ks], sf[cg][ks], ks > 0 ? acc[rg][cg] : PASS == 1 ? zero : init[rg], 0, 0, 0);
            };
            auto epilogue = [&](int rb) {
                if (mask) {      // a scalar branch
                    const int t = lane_again();
                    int sP[4];
#pragma unroll
                    for (int cg = 0; cg < 4; ++cg) sP[cg] = sparse ? spos[cg * 256 + wave * 64 + t] : w0 + 16 * cg + (t & 15);
                    mask_block<PASS>(acc, x0 + rb * 32 + 4 * (t >> 4), sP);   // streamed index of entry i of acc[rg][.]: + 16*rg + i
                }
                if (PASS == 1) lse_block_epilogue(acc, scale2, m, l);
                else colsum_block_epilogue(acc, scale2, run);
            };
            multiply();
            __builtin_amdgcn_sched_barrier(0);
            fetch(cur, 1);
            if (PASS == 2) fetch_init(cur_l, 1);
            __builtin_amdgcn_sched_barrier(0);
            epilogue(0);
            __builtin_amdgcn_sched_barrier(0);
            multiply();
            __builtin_amdgcn_sched_barrier(0);
            finish_tile();
            __builtin_amdgcn_sched_barrier(0);
            epilogue(1);
            __builtin_amdgcn_sched_barrier(0);
        } else {
            finish_tile();
        }
    };
    for (int it = 0; it < n_it; it += 2) {
        tile_step(std::integral_constant<int, 0>{}, it);
        if (it + 1 < n_it) tile_step(std::integral_constant<int, 1>{}, it + 1);
    }

    // fold the four lanes (equal c16) that share a stationary row - the pairs (q4, q4 ^ 1) first, lower lane first,
    // then the two pairs - and write the chunk's partial for rows 0..255 of the strip
    float* pa = part_a + ((size_t)h * n_chunks_total * nSp + u) * BS;
    float* pb = part_b + ((size_t)h * n_chunks_total * nSp + u) * BS;
#pragma unroll
    for (int cg = 0; cg < 4; ++cg) {
        const int r = wave * 64 + cg * 16 + c16;
        if (PASS == 1) {
            float mm = m[cg], ll = l[cg];
#pragma unroll
            for (int step = 16; step <= 32; step <<= 1) {     // (only the lower lane of a pair is read from here on)
                const float mo = __shfl_xor(mm, step), lo = __shfl_xor(ll, step);
                const float M = fmaxf(mm, mo);
                ll = ll * __builtin_amdgcn_exp2f(mm - M) + lo * __builtin_amdgcn_exp2f(mo - M);
                mm = M;
            }
            if (q4 == 0) { pa[r] = mm; pb[r] = ll; }
        } else {
            float v = run[cg];
#pragma unroll
            for (int step = 16; step <= 32; step <<= 1) v += __shfl_xor(v, step);
            if (q4 == 0) pa[r] = v;
        }
    }
}

// Folds the chunks of every strip, in chunk order: pass 1 -> lse2[h, i] = log2 sum_j 2^(c q_i.k_j) per query
// head; pass 2 -> scores[h, j] = A_s[j] per key head, the partials of its `group` query heads added in head
// order (group = 1: one query head per key head).  One thread per (head, row).  With key lists (pass 2 over the
// competing keys only) row r of strip t is the list's entry t * 256 + r and its score goes to that key's
// position; the workgroups of the grid from nS on then write the inverse norms of the PROTECTED keys, which
// pass 2 no longer holds (summed in the order of the stand-alone norm kernel, so all three give the same bits).
template <int PASS>
__global__ void __launch_bounds__(256)
k_score_combine(int group, int L, int R0, int C, const float* __restrict__ part_a, const float* __restrict__ part_b,
                float* __restrict__ out, const int32_t* __restrict__ lists, const bf16_t* __restrict__ k,
                float* __restrict__ rnorm, int nS)
{
    const int h = blockIdx.y, r = threadIdx.x;
    int tile = blockIdx.x;
    if (PASS == 2 && lists != nullptr && tile >= nS) {
        if (rnorm != nullptr) protected_norms(lists, h, L, k, rnorm, (tile - nS) * 32 + (r >> 3), 32 * ((int)gridDim.x - nS));
        return;
    }
    const bool sparse = PASS == 2 && lists != nullptr;
    int row = tile * BS + r;
    const int CT = C * BX, G = (L + CT - 1) / CT;
    int g0 = first_chunk(PASS, tile, CT, R0), nc = strip_chunks(PASS, tile, L, CT, R0);
    if (sparse) {
        // what the lists say, in one memory latency: entries past the end of the list hold anything
        const int in_list = row, rows = lists[0], p_strip = lists[LIST_HEAD + tile * BS];
        row = lists[LIST_HEAD + min(in_list, L - 1)];
        if (in_list >= rows) return;
        g0 = sparse_first_chunk(p_strip, R0, CT);
        nc = G - g0;
    } else if (row >= L) return;
    if (nc == 0) return;     // pass 1 under a window: a strip with no row that counts (its values are never read)
    const int t_base = (PASS == 1) ? R0 / BS : 0, nSp = nS - t_base;   // as in k_score_mfma
    const size_t stride = (size_t)nSp * BS;     // from one chunk of a strip to the next
    const int h_first = (PASS == 1) ? h : h * group;      // first query head whose partials are read
    const float* pa = part_a + (((size_t)h_first * G + g0) * nSp + (tile - t_base)) * BS + r;
    const float* pb = part_b + (((size_t)h_first * G + g0) * nSp + (tile - t_base)) * BS + r;
    // Eight chunks at a time, all loads in flight together: chunks past the last one are read as the last one and left out.  (A
    // loop over the chunks takes its remainder one memory latency after the other, which is most of a kernel that lives for
    // 5 us: timed with events, folds of pass 1 for 32 heads x 2896 8.4 -> 6.5 us, x 12644 10.3 -> 7.5, of pass 2 for 32 query
    // heads on 8 key heads x 6144 11.5 -> 7.3.)
    constexpr int AHEAD = 8;
    if (PASS == 1) {
        float M = -1e30f, Ls = 0.f;
        auto fold = [&](auto ahead) {
            constexpr int N = decltype(ahead)::value;
            float a[N], b[N];
            for (int c0 = N; c0 < nc; c0 += N) {             // the largest reference of all chunks before any sum, so that none is rescaled
#pragma unroll
                for (int i = 0; i < N; ++i) a[i] = pa[(size_t)min(c0 + i, nc - 1) * stride];
#pragma unroll
                for (int i = 0; i < N; ++i) M = fmaxf(M, a[i]);
            }
            for (int c0 = 0; c0 < nc; c0 += N) {
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const size_t at = (size_t)min(c0 + i, nc - 1) * stride;
                    a[i] = pa[at];
                    b[i] = pb[at];
                }
                if (c0 == 0)
#pragma unroll
                    for (int i = 0; i < N; ++i) M = fmaxf(M, a[i]);
#pragma unroll
                for (int i = 0; i < N; ++i)
                    if (c0 + i < nc) Ls = fmaf(b[i], exp2f(a[i] - M), Ls);
            }
        };
        if (nc <= AHEAD) fold(std::integral_constant<int, AHEAD>{});
        else fold(std::integral_constant<int, 2 * AHEAD>{});         // (more than one round trip costs a second one for the references)
        out[(size_t)h * L + row] = M + log2f(Ls);
    } else {
        float sum = 0.f;
        if (group == 1) {
            for (int c0 = 0; c0 < nc; c0 += AHEAD) {
                float a[AHEAD];
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) a[i] = pa[(size_t)min(c0 + i, nc - 1) * stride];
#pragma unroll
                for (int i = 0; i < AHEAD; ++i)
                    if (c0 + i < nc) sum += a[i];
            }
        } else {                                             // chunk by chunk of one query head after the other
            const int terms = group * nc;
            int m = 0, c = 0;
            for (int t0 = 0; t0 < terms; t0 += AHEAD) {
                float a[AHEAD];
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) {
                    a[i] = pa[((size_t)m * G + c) * stride];
                    if (t0 + i + 1 < terms && ++c == nc) { c = 0; ++m; }
                }
#pragma unroll
                for (int i = 0; i < AHEAD; ++i)
                    if (t0 + i < terms) sum += a[i];
            }
        }
        out[(size_t)h * L + row] = sum;
    }
}

}  // namespace lookm

namespace lookm_host {

// Tiles per chunk.  Short chunks waste the start-up of their workgroups (the stationary rows, the first tile: 4 us or
// so, only partly hidden by the two others of the compute unit) and the fold's time; long ones leave a few rounds of
// workgroups and an uneven last one.  Both passes with their folds, event-free kernel times in us:
//   total tiles (heads x length)      C =  1     2     3     4     6     8    12    16    20    24    40
//      168  (8 x 700)                     26    28    31    33    39    45    53    53
//      672  (8 x 1482)                    39    34    34    35    40    45    56    67
//     2304  (8 x 2896)                    82    61    54    50    51    56    59    69
//     9.2 K (32 x 2896)                                    118   115   118   115   116   132   140   171
//    20 K   (8 x 8871)                   504   290   250   227   210   199   197   197
//    45 K   (40 x 5904)                                    419   391   383   361   373   361   379   393
//   160 K   (32 x 12644)                                  1377  1245  1194  1147  1139  1124  1126  1131
//   264 K   (8 x 32768)                                   2551  2166  2012  1916  1884  1850  1843  1831
//    1.06 M (32 x 32768)                    C = 40: 7239   67: 7212   100: 7227   172: 7252
//    4.23 M (128 x 32768)                                133: 28570   256: 28900
// The best length grows like the square root of the total.
static long all_tiles(int H, int L)
{
    long total = 0;
    const int nS = (L + lookm::BS - 1) / lookm::BS;
    for (int t = 0; t < nS; ++t) total += (L - t * lookm::BS + lookm::BX - 1) / lookm::BX;
    return total * H;
}
static int chunk_tiles(int H, int L) { return std::max(1, (int)std::ceil(0.065 * std::sqrt((double)all_tiles(H, L)))); }
// The chunk length whose partials every workspace holds: a smaller workspace than lookm_workspace_bytes gives is accepted
// down to this, so that the sizes that a program has kept, or taken from its longest prompt, stay good for short chunks too.
static int roomy_chunk_tiles(int H, int L)
{
    return (int)std::min(256l, std::max(8l, (all_tiles(H, L) + 6143) / 6144));
}

// floats of the chunk partials: two arrays [H][chunks][strips][256]
static size_t partial_floats(int H, int L, int C)
{
    const int nS = (L + lookm::BS - 1) / lookm::BS, G = (L + C * lookm::BX - 1) / (C * lookm::BX);
    return (size_t)2 * H * G * nS * lookm::BS;
}

static int total_chunks(int pass, int L, int C, int R0)
{
    const int nS = (L + lookm::BS - 1) / lookm::BS;
    int u = 0;
    for (int t = 0; t < nS; ++t) u += lookm::strip_chunks(pass, t, L, C * lookm::BX, R0);
    return u;
}

// workgroups of one score pass: 8 XCD lanes x (units per lane), see the mapping at the top of k_score_mfma
static unsigned score_grid(int H, int U)
{
    if (H >= 8) return 8u * (unsigned)((H + 7) / 8) * (unsigned)U;
    const int xph = 8 / H;
    return 8u * (unsigned)((U + xph - 1) / xph);
}

size_t scores_mfma_scratch_floats(int H, int L, bool least)
{
    const size_t floor = partial_floats(H, L, roomy_chunk_tiles(H, L));
    return least ? floor : std::max(floor, partial_floats(H, L, chunk_tiles(H, L)));
}

// mask / M / lists: when given (the caller does not want the scores of the protected keys), pass 2 runs over the
// competing keys only; lists: device, 2 * L + LIST_HEAD ints
int launch_scores_mfma(const void* q, const void* k, int H, int kv_heads, int L, int d, int R0, float* lse,
                       const float* lse_in, float* scores, float* rnorm, float* scratch, size_t scratch_floats,
                       const uint8_t* mask, int M, int32_t* lists, ScoreParts* parts, hipStream_t st)
{
    if (d != lookm::SD) return LOOKM_ERR_UNSUPPORTED;
    const LaunchCheck check;
    const int group = H / kv_heads;
    const int nS = (L + lookm::BS - 1) / lookm::BS;
    int C = chunk_tiles(H, L);
    while (partial_floats(H, L, C) > scratch_floats) ++C;      // (ends: roomy_chunk_tiles' partials fit)
    const int G = (L + C * lookm::BX - 1) / (C * lookm::BX);
    // Pass 2 keeps the full problem's chunk length also under a window (its partial arrays keep their layout).
    // Pass 1 under a window runs only the last strips, each over all keys: shorter chunks give the chip enough
    // workgroups, as far as the partial arrays (sized for the full problem) hold them.
    int C1 = C;
    if (R0 > 0) {
        const int nS1 = nS - R0 / lookm::BS;
        const long want = (long)nS1 * ((L + lookm::BX - 1) / lookm::BX) * H / 2048;   // tiles per chunk for ~2048 units
        C1 = (int)std::min<long>(C, std::max<long>(4, want));
        while (C1 < C && (long)((L + C1 * lookm::BX - 1) / (C1 * lookm::BX)) * nS1 > (long)G * nS) ++C1;
    }
    const int U1 = total_chunks(1, L, C1, R0), U2 = total_chunks(2, L, C, R0);
    float* part_a = scratch;
    float* part_b = scratch + (size_t)H * G * nS * lookm::BS;
    const float scale2 = lookm::kLog2e / sqrtf((float)d);
    const lookm::bf16_t* qq = (const lookm::bf16_t*)q;
    const lookm::bf16_t* kk = (const lookm::bf16_t*)k;
    const bool sparse = mask != nullptr && lists != nullptr;
    if (!lse_in) {
        // with a mask the launch has one workgroup more: it builds the key lists while the others compute
        hipLaunchKernelGGL((lookm::k_score_mfma<1, false>), dim3(score_grid(H, U1) + (sparse ? 1u : 0u)), dim3(256), 0, st, qq, kk, H,
                           group, L, R0, scale2, C1, U1, lse, 1.0f, part_a, part_b, (float*)nullptr,
                           sparse ? mask : (const uint8_t*)nullptr, M, lists);
        mark(LOOKM_K_SCORE_LSE);
        hipLaunchKernelGGL(lookm::k_score_combine<1>, dim3(nS, H), dim3(256), 0, st, 1, L, R0, C1, part_a, part_b, lse,
                           (const int32_t*)nullptr, (const lookm::bf16_t*)nullptr, (float*)nullptr, nS);
        mark(LOOKM_K_SCORE_LSE_FOLD);
    } else if (sparse) {
        hipLaunchKernelGGL(lookm::k_score_lists, dim3(1), dim3(1024), 0, st, mask, L, M, lists);
    }
    // a caller-supplied row log-sum-exp is natural-log: one factor log2(e) brings it to the kernels' base
    if (sparse)
        hipLaunchKernelGGL((lookm::k_score_mfma<2, true>), dim3(score_grid(H, U2)), dim3(256), 0, st, qq, kk, H, group, L,
                           R0, scale2, C, U2, lse_in ? lse_in : lse, (lse_in ? lookm::kLog2e : 1.0f) / scale2, part_a,
                           part_b, rnorm, (const uint8_t*)nullptr, M, lists);
    else
        hipLaunchKernelGGL((lookm::k_score_mfma<2, false>), dim3(score_grid(H, U2)), dim3(256), 0, st, qq, kk, H, group, L,
                           R0, scale2, C, U2, lse_in ? lse_in : lse, (lse_in ? lookm::kLog2e : 1.0f) / scale2, part_a,
                           part_b, rnorm, (const uint8_t*)nullptr, M, (int32_t*)nullptr);
    mark(LOOKM_K_SCORE_COLSUM);
    // Short prompts: the selection sums the chunks itself, a kernel less (see k_select).  Up to sixteen chunks, two round trips, where
    // it has 512 threads at most, up to eight, one, where it has 1024: beyond, a single workgroup a head reads for longer than the
    // launch costs.  Whole layers, us, with the fold's kernel / summed there: one head x 1024 (16 chunks), nearly all images 43.3 / 42.8, half
    // text 50.6 / 48.3; two heads x 1024 47.5 / 46.8; one head, nearly all images, x 1088 (17 chunks) 48.8 / 49.8, x 1344 (21) 51.2 / 52.0,
    // x 2048 (32) 59.8 / 60.8, two x 1088 49.4 / 50.3, x 1600 (25) 54.5 / 56.0; 1024
    // threads: 8 heads x 2896 in twelve chunks 72.7 / 73.1, one head x 2428 in nineteen 57.9 / 61.2.  Workgroups of 1024 threads, two to a
    // compute unit, are also a slow way through many norms once the heads' own ones are on every compute unit: x 2100, most of it text, 128
    // heads 278.3 / 273.6, 192 386.2 / 383.5, 256 490.8 / 498.2, x 3144 760 / 772.
    // (H: the heads' workgroups and those of the norms are one grid.)
    if (parts && sparse && group == 1 && L <= SELECT_SUMS_MAX_L && (L <= 2048 ? G <= 16 && H <= 4096 : G <= 8 && H <= 192)) {
        parts->part = part_a;
        parts->lists = lists;
        parts->k = k;
        parts->rnorm = rnorm;
        parts->CT = C * lookm::BX;
        parts->G = G;
        parts->R0 = R0;
        return check.status();
    }
    // Workgroups for the norms of the protected keys: as many as strips.  Few heads of up to 2048 tokens: up to four times as many, with
    // which eight threads have two keys at most instead of eight (one head x 1344, half text, 58.4 -> 56.4 us the whole layer, 57.2
    // in the selection; x 2048 with 1472 text tokens 60.6 -> 57.4, 58.6; 2 x 1600, nearly all images, 54.4 -> 54.6, 55.9) - one a
    // compute unit in all: 800 workgroups that find no key more, 128 query heads on 32 x 1748, nearly all images, 6.5 -> 8.3 us.
    const int norm_blocks = !sparse ? 0 : L > 2048 ? nS : std::min(4 * nS, std::max(nS, 256 / kv_heads - nS));
    hipLaunchKernelGGL(lookm::k_score_combine<2>, dim3(nS + norm_blocks, kv_heads), dim3(256), 0, st, group, L, R0, C,
                       part_a, part_b, scores, sparse ? (const int32_t*)lists : (const int32_t*)nullptr, kk, rnorm, nS);
    mark(LOOKM_K_SCORE_COLSUM_FOLD);
    return check.status();
}

}  // namespace lookm_host
