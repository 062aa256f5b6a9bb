// Text-prior selection (Section 3.2, Eq. 5-8): one workgroup per head.
//
// Protected positions (text tokens, and the last M positions of any modality) are always
// conserved; the remaining budget k_img = B - |protected| goes to the image positions outside the
// window with the highest accumulated score.  Eq. 5's "add max(A_s) to text scores" only serves to
// rank every text token above every image token, so it is realised as a class, not as a float add.
// The k_img-th largest score is found by an MSB-first radix select over the monotone integer image
// of the float bits, re-based to the head's own range (an LDS histogram over a digit of 10 to 12 bits; the few keys that
// share the threshold's digit are then ranked against each other directly, or, if they are many, by further
// digits); equal scores are resolved towards the lower position by an ordered prefix
// count.  Kept and evicted index lists come out ascending.
// Supports L <= 32 * 1024 (32 positions per thread).
#include "score_parts.h"

#include <type_traits>

namespace lookm {

constexpr int SEL_CAND = 4096;    // capacity of the LDS candidate list
constexpr int SEL_FAST = 128;     // up to this many candidates are ranked all against all

// order-preserving map float -> uint32 (larger float <=> larger key); -0 is folded onto +0
__device__ __forceinline__ uint32_t score_key(float s)
{
    uint32_t b = __float_as_uint(s);
    if (b == 0x80000000u) b = 0u;
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// exclusive prefix sum over the workgroup's WAVES waves of one wave-uniform int, and the total.  One barrier;
// `wtot` is an LDS array that nothing else touches (every scan of the kernel has its own).
template <int WAVES>
__device__ __forceinline__ int wave_scan_excl(int wave_value, int* wtot, int& total)
{
    const int wave = threadIdx.x >> 6;
    if (lane_id() == 0) wtot[wave] = wave_value;
    __syncthreads();
    int before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const int c = wtot[w];
        before += (w < wave) ? c : 0;
        tot += c;
    }
    total = tot;
    return before;
}

// Wave w owns the contiguous segment [w*64*IPT, (w+1)*64*IPT) of positions; inside it lane l holds
// positions seg + i*64 + l, i < IPT, so global reads and writes are coalesced.  Keys and classes are
// read once and stay in registers for the radix passes and the compaction; ordered counts are ballots
// inside the wave plus one 16-entry scan across waves.
//
// SUMS (short prompts, bf16 x 128): the scores of the competing tokens arrive as the score pass' partials per chunk of query
// rows, and every thread adds up those of its own positions, in the order of k_score_combine.  Competing tokens are numbered as in
// the pass: by an ordered count.  Workgroups past the H heads compute the inverse norms of the protected keys, which that
// kernel does otherwise.  A launch and a round trip less, for a barrier and a longer load.  Whole layers, us, summed by a kernel of
// its own / here: 8 heads x 676 47.1 / 45.5, 32 x 876 63.4 / 60.7, 32 x 1482 78.0 / 76.5, 40 x 2228 130.4 / 128.9, 32 x 4056 with
// a row log-sum-exp 150.2 / 148.2 (32 x 2896: fold and selection 4.8 + 7.0 / 10.6, without the gap between the two).
template <int IPT, int SEL_THREADS, bool SUMS>
__global__ void __launch_bounds__(SEL_THREADS)
k_select(const float* __restrict__ scores, lookm_host::ScoreParts parts, int H, int norm_blocks, const uint8_t* __restrict__ mask,
         int L, int B, int M, int rule, int32_t* __restrict__ kept, int32_t* __restrict__ evicted, int32_t* __restrict__ status)
{
    constexpr int SEL_WAVES = SEL_THREADS / 64;
    constexpr int DIGIT = (SEL_THREADS == 1024) ? 12 : (SEL_THREADS == 512) ? 11 : 10, SEL_BINS = 1 << DIGIT;    // four bins a thread
    static_assert(SEL_BINS == 4 * SEL_THREADS, "");
    __shared__ int hist[SEL_BINS];
    __shared__ uint32_t cand[SEL_CAND];     // keys that share the threshold's first digit
    __shared__ int wtot[8][SEL_WAVES];      // one row per workgroup-wide scan
    __shared__ uint32_t wmin[SEL_WAVES], wmax[SEL_WAVES], wtmin[SEL_WAVES], wtmax[SEL_WAVES];
    __shared__ int sh_bin, sh_k, sh_ncand;
    __shared__ uint32_t sh_thr;

    const int h = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    if (SUMS && h >= H) {
        const int u = h - H;
        protected_norms(parts.lists, u / norm_blocks, L, static_cast<const bf16_t*>(parts.k), parts.rnorm,
                        (u % norm_blocks) * (SEL_THREADS / 8) + (tid >> 3), norm_blocks * (SEL_THREADS / 8));
        return;
    }
    if (!SUMS) scores += (size_t)h * L;
    kept += (size_t)h * B;
    evicted += (size_t)h * (L - B);
    const int head_len = L - M;   // positions [0, head_len) are outside the recent window
    const int seg = wave * 64 * IPT;

    // every load is issued before the first use, so the whole read costs one memory latency
    uint32_t key[IPT];
    uint8_t img[IPT];
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const int jc = min(seg + i * 64 + lane, L - 1);   // unconditional loads of a clamped index: nothing waits on a branch
        key[i] = SUMS ? 0u : __float_as_uint(scores[jc]);
        img[i] = mask[jc];
    }
    for (int i = tid; i < SEL_BINS; i += SEL_THREADS) hist[i] = 0;
    if (tid == 0) sh_ncand = 0;
    if constexpr (SUMS) {
        uint64_t comp[IPT];                      // competing positions of the wave's rows
        int n = 0, all;
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            comp[i] = __ballot(img[i] != 0 && seg + i * 64 + lane < head_len);
            n += __popcll(comp[i]);
        }
        n = wave_scan_excl<SEL_WAVES>(n, wtot[5], all);
        const int nS = (L + BS - 1) / BS;
        const size_t stride = (size_t)nS * BS;
        int at[IPT], g0[IPT];
        float sum[IPT];
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            at[i] = min(n + mask_rank(comp[i]), L - 1);       // number among the competing tokens
            n += __popcll(comp[i]);
            g0[i] = sparse_first_chunk(parts.lists[LIST_HEAD + (at[i] / BS) * BS], parts.R0, parts.CT);
            sum[i] = 0.f;
        }
        const float* part = parts.part + (size_t)h * parts.G * stride;
        for (int g = 0; g < parts.G; g += 8) {                // eight chunks of all positions in flight
            float x[IPT][8];
#pragma unroll
            for (int i = 0; i < IPT; ++i)
#pragma unroll
                for (int c = 0; c < 8; ++c) x[i][c] = part[min(g + c, parts.G - 1) * stride + at[i]];
#pragma unroll
            for (int i = 0; i < IPT; ++i)
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    if (g + c >= g0[i] && g + c < parts.G) sum[i] += x[i][c];      // (below: not the strip's, never written)
        }
#pragma unroll
        for (int i = 0; i < IPT; ++i) key[i] = __float_as_uint(sum[i]);
    }

    // bit i of each mask: position seg + i*64 + lane is in the recent window / a text token before it / an image
    // token before it
    uint32_t win_m = 0, text_m = 0, img_m = 0;
    uint32_t kmin = 0xffffffffu, kmax = 0u;       // over the image tokens before the window
    uint32_t tmin = 0xffffffffu, tmax = 0u;       // over the text tokens before the window (literal rule only)
    int ntext_wave = 0;
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const int j = seg + i * 64 + lane;
        bool text = false;
        if (j < L) {
            key[i] = score_key(__uint_as_float(key[i]));
            if (j >= head_len) win_m |= 1u << i;
            else if (img[i] == 0) {
                text = true;
                text_m |= 1u << i;
                if (rule == LOOKM_SELECT_LITERAL) { tmin = min(tmin, key[i]); tmax = max(tmax, key[i]); }
            } else {
                img_m |= 1u << i;
                kmin = min(kmin, key[i]);
                kmax = max(kmax, key[i]);
            }
        }
        ntext_wave += __popcll(__ballot(text));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, off));
        kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, off));
    }
    if (rule == LOOKM_SELECT_LITERAL) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            tmin = min(tmin, (uint32_t)__shfl_xor((int)tmin, off));
            tmax = max(tmax, (uint32_t)__shfl_xor((int)tmax, off));
        }
    }
    if (lane == 0) { wmin[wave] = kmin; wmax[wave] = kmax; wtmin[wave] = tmin; wtmax[wave] = tmax; }

    int ntext;   // text tokens before the window; |T u R| = ntext + M
    wave_scan_excl<SEL_WAVES>(ntext_wave, wtot[0], ntext);
    const int nprot = ntext + M;
    // Eq. 8 has N = B - M places before the window.  If they hold every text token, text and window are sure and
    // the image tokens compete for the rest; if not, the default rule reports an error, while the literal rule
    // lets the (boosted, hence always higher-ranked) text tokens compete for the N places and conserves no image.
    const bool text_competes = (B < nprot) && (rule == LOOKM_SELECT_LITERAL);
    if (B < nprot && !text_competes) {
        // text + window do not fit: report, and leave in-range (meaningless) index lists behind
        if (tid == 0) *status = LOOKM_ERR_BUDGET_BELOW_PROTECTED;
        for (int r = tid; r < B; r += SEL_THREADS) kept[r] = r;
        for (int e = tid; e < L - B; e += SEL_THREADS) evicted[e] = B + e;
        return;
    }
    if (tid == 0 && h == 0) *status = LOOKM_OK;
    const uint32_t prot_m = text_competes ? win_m : (win_m | text_m);   // conserved whatever the scores
    const uint32_t evic_m = text_competes ? text_m : img_m;             // compete by score
    const int k_img = text_competes ? B - M : B - nprot;                // places they compete for
    const int n_evictable = text_competes ? ntext : L - nprot;
    kmin = 0xffffffffu;
    kmax = 0u;
#pragma unroll
    for (int w = 0; w < SEL_WAVES; ++w) {
        kmin = min(kmin, text_competes ? wtmin[w] : wmin[w]);
        kmax = max(kmax, text_competes ? wtmax[w] : wmax[w]);
    }
    // Scores of a head crowd into a few binades, so the raw top bits would send most keys to a handful of
    // histogram bins.  Keys are re-based to the competing tokens' own range [kmin, kmax] and shifted up to use
    // all 32 bits: order and equality are unchanged, the first digit spreads over the bins, and few keys are
    // left to tell apart after it.
    {
        const uint32_t range = (kmax >= kmin) ? kmax - kmin : 0u;
        const int lz = range ? __clz(range) : 0;
#pragma unroll
        for (int i = 0; i < IPT; ++i) key[i] = (key[i] - kmin) << lz;   // only competing entries are used below
    }
    const bool keep_all = (k_img == n_evictable), keep_none = (k_img == 0);

    // key of the k_img-th largest evictable score, and how many keys equal to it to take
    uint32_t thr = 0;
    int need_eq = 0;
    if (!keep_all && !keep_none) {
        int kk = k_img;
        int scan_row = 1;
        // finds the bin (counting from the top) where the running count first reaches kk; every thread
        // owns up to four consecutive bins in descending order.  Two barriers.
        auto find_bin = [&](int nbins) {
            const int per = (nbins + SEL_THREADS - 1) / SEL_THREADS;   // 4 or 1
            int c[4] = {0, 0, 0, 0}, sum = 0;
            for (int i = 0; i < per; ++i) {
                const int bin = nbins - 1 - (tid * per + i);
                c[i] = (bin >= 0) ? hist[bin] : 0;
                sum += c[i];
            }
            int incl = sum;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int v = __shfl_up(incl, off);
                if (lane >= off) incl += v;
            }
            int tot;
            int cum = wave_scan_excl<SEL_WAVES>(__shfl(incl, 63), wtot[scan_row++], tot) + incl - sum;   // count in bins above mine
            for (int i = 0; i < per; ++i) {
                if (cum < kk && cum + c[i] >= kk) { sh_bin = nbins - 1 - (tid * per + i); sh_k = kk - cum; }
                cum += c[i];
            }
            __syncthreads();
            kk = sh_k;
            return (uint32_t)sh_bin;
        };

#pragma unroll
        for (int i = 0; i < IPT; ++i)
            if ((evic_m >> i) & 1u) atomicAdd(&hist[key[i] >> (32 - DIGIT)], 1);   // hist was cleared before the first barrier
        __syncthreads();
        const uint32_t d0 = find_bin(SEL_BINS);
        const int n_cand = hist[d0];
        const bool listed = n_cand <= SEL_CAND;
        if (listed) {
#pragma unroll
            for (int i = 0; i < IPT; ++i)
                if (((evic_m >> i) & 1u) && (key[i] >> (32 - DIGIT)) == d0) cand[atomicAdd(&sh_ncand, 1)] = key[i];
        }
        __syncthreads();
        if (n_cand <= SEL_FAST) {
            // few candidates: each is compared with all the others (the list is read as LDS broadcasts)
            if (tid < n_cand) {
                const uint32_t mine = cand[tid];
                int above = 0, same = 0;
                for (int c = 0; c < n_cand; ++c) {
                    const uint32_t x = cand[c];
                    above += (x > mine) ? 1 : 0;
                    same += (x == mine) ? 1 : 0;
                }
                if (above < kk && kk <= above + same) { sh_thr = mine; sh_k = kk - above; }
            }
            __syncthreads();
            thr = sh_thr;
            need_eq = sh_k;
        } else {
            // many keys share the first digit: further digits, over the LDS list, or over the registers when even the list
            // is too small
            thr = d0;
#pragma unroll
            for (int done = DIGIT; done < 32; done += DIGIT) {
                const int width = min(DIGIT, 32 - done), shift = 32 - done - width;
                for (int i = tid; i < 1 << width; i += SEL_THREADS) hist[i] = 0;
                __syncthreads();
                auto count = [&](uint32_t x) {
                    if ((x >> (32 - done)) == thr) atomicAdd(&hist[(x >> shift) & ((1u << width) - 1u)], 1);
                };
                if (listed) {
                    for (int c = tid; c < n_cand; c += SEL_THREADS) count(cand[c]);
                } else {
#pragma unroll
                    for (int i = 0; i < IPT; ++i)
                        if ((evic_m >> i) & 1u) count(key[i]);
                }
                __syncthreads();
                thr = (thr << width) | find_bin(1 << width);
            }
            need_eq = kk;
        }
    }

    // ordered compaction.  Keys above the threshold and protected positions are conserved; of the keys equal
    // to it, those at the lowest positions fill what is left.  One scan carries both counts.
    uint32_t keep_m = prot_m, eq_m = 0;
    int sure_wave = 0, eq_wave = 0;
    if (keep_all) keep_m |= evic_m;
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        bool eq = false;
        if (!keep_all && !keep_none && ((evic_m >> i) & 1u)) {
            if (key[i] > thr) keep_m |= 1u << i;
            else if (key[i] == thr) { eq = true; eq_m |= 1u << i; }
        }
        eq_wave += __popcll(__ballot(eq));
        sure_wave += __popcll(__ballot((keep_m >> i) & 1u));
    }
    if (lane == 0) { wtot[6][wave] = sure_wave; wtot[7][wave] = eq_wave; }
    __syncthreads();
    int sure_before = 0, eq_run = 0;
#pragma unroll
    for (int w = 0; w < SEL_WAVES; ++w) {
        sure_before += (w < wave) ? wtot[6][w] : 0;
        eq_run += (w < wave) ? wtot[7][w] : 0;
    }
    int kp = sure_before + min(eq_run, need_eq);           // conserved positions in lower waves
    int ep = min(seg, L) - kp;                              // evicted positions in lower waves
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const bool eq = (eq_m >> i) & 1u;
        const uint64_t eb = __ballot(eq);
        if (eq && eq_run + mask_rank(eb) < need_eq) keep_m |= 1u << i;
        eq_run += __popcll(eb);
        const int j = seg + i * 64 + lane;
        const bool valid = j < L, keep = (keep_m >> i) & 1u;
        const uint64_t kb = __ballot(valid && keep), vb = __ballot(valid);
        if (valid) {
            const int r = mask_rank(kb);
            if (keep) kept[kp + r] = j;
            else evicted[ep + lane - r] = j;               // valid lanes are a prefix of the wave
        }
        kp += __popcll(kb);
        ep += __popcll(vb) - __popcll(kb);
    }
}

}  // namespace lookm

namespace lookm_host {

int launch_select(const float* scores, const ScoreParts& parts, const uint8_t* mask, int H, int L, int budget, int M, int rule, int32_t* kept,
                  int32_t* evicted, int32_t* status, hipStream_t st)
{
    const LaunchCheck check;
    auto go = [&](auto ipt, auto threads) {
        constexpr int IPT = decltype(ipt)::value, THREADS = decltype(threads)::value;
        if constexpr (IPT * THREADS <= SELECT_SUMS_MAX_L)
            if (parts.part != nullptr) {
                const int norm_blocks = (L + THREADS / 2 - 1) / (THREADS / 2);            // up to four keys for eight threads
                hipLaunchKernelGGL((lookm::k_select<IPT, THREADS, true>), dim3(parts.rnorm ? H + H * norm_blocks : H), dim3(THREADS), 0, st, scores,
                                   parts, H, norm_blocks, mask, L, budget, M, rule, kept, evicted, status);
                return;
            }
        hipLaunchKernelGGL((lookm::k_select<IPT, THREADS, false>), dim3(H), dim3(THREADS), 0, st, scores, parts, H, 0, mask, L, budget, M, rule,
                           kept, evicted, status);
    };
#define LOOKM_SELECT(ipt, threads) go(std::integral_constant<int, ipt>{}, std::integral_constant<int, threads>{})
    // Barriers and scans across sixteen waves cost more than a short prompt's positions.  32 heads, us with 1024 / 512 / 256
    // threads: 256 positions 5.5 / 4.3 / 4.2, 512 5.5 / 4.5 / 4.5, 1024 5.7 / 5.0 / 5.2, 2048 6.4 / 5.8 / 6.7,
    // 2800 7.2 / 7.6 / 9.9 (back-to-back calls; four positions a thread at least, as before, 6.5, 6.6, 6.7, 7.0).
    if (L <= 256) LOOKM_SELECT(1, 256);
    else if (L <= 512) LOOKM_SELECT(1, 512);
    else if (L <= 1024) LOOKM_SELECT(2, 512);
    else if (L <= 2048) LOOKM_SELECT(4, 512);
    else if (L <= 4096) LOOKM_SELECT(4, 1024);
    else if (L <= 8192) LOOKM_SELECT(8, 1024);
    else if (L <= 16384) LOOKM_SELECT(16, 1024);
    else if (L <= 32768) LOOKM_SELECT(32, 1024);
    else
        return LOOKM_ERR_UNSUPPORTED;
#undef LOOKM_SELECT
    mark(LOOKM_K_SELECT);
    return check.status();
}

}  // namespace lookm_host
