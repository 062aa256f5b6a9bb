// KV-pair merging and compaction (Section 3.3, Eq. 10-12; layout of Eq. 6-7).
//
// k_bucket groups the evicted tokens of a head by the conserved slot they were matched to (the
// paper's one-to-many similarity sets k_sim), as a stable counting sort so that every set lists its
// members' positions (with their matching cosines) in ascending position.  k_merge then GATHERS: a workgroup
// reads the rows of some consecutive conserved slots and those of all their members and writes the compact output
// rows - no scatter, no float atomics, fixed summation order, coalesced 16-byte accesses along the head
// dimension.  Keys and values use the same sets and (for weighted merging) the same cosine weights.
// Short lists are not sorted beforehand: the merge's workgroups collect their slots' members from the assignment list
// (collect_members), for the shortest ones every wave by itself (k_merge_direct).
#include "common.h"

#include <algorithm>

namespace lookm {

constexpr int BK_THREADS = 1024;
constexpr int BK_WAVES = BK_THREADS / 64;
constexpr int BK_MAX_SEG = 1024;   // slots per workgroup: 16 counter rows of this many ints, and the entry lists, fit in LDS

// lanes of the wave whose (valid) key equals this lane's key
__device__ __forceinline__ uint64_t match_key(int key, bool valid, int nbits)
{
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < nbits; ++b) {
        const bool bit = (key >> b) & 1;
        const uint64_t m = __ballot(bit && valid);
        peers &= bit ? m : ~m;
    }
    return peers;
}

// One workgroup per (head, segment of S consecutive conserved slots); the segments of a head run on
// different compute units.  Every workgroup reads the head's whole assignment list once - each thread its IPT
// entries, all loads in flight together - counts the entries matched to slots below its segment (that is
// where its part of the member lists starts) and sorts the entries matched to its own slots: wave w owns
// entries [w*64*IPT, (w+1)*64*IPT), lane l holds entries seg + i*64 + l.  The wave first compacts its own
// entries into an LDS list, in order, so that the ranking below runs over full 64-lane rows of entries that
// matter rather than over rows where most lanes belong to other segments.  Counts per (wave, slot) are turned
// into start offsets in slot-major, wave-minor order, which makes the fill stable across waves; inside a wave
// the list is taken 64 entries at a time and lanes with equal slots are ranked by lane.
//
// It also writes where every slot's members begin, first[0 .. B] for a head, first[B] = Le.
template <int IPT>
__global__ void __launch_bounds__(BK_THREADS)
k_bucket(const int32_t* __restrict__ assign, const int32_t* __restrict__ evicted, const float* __restrict__ sim,
         int Le, int B, int S, int nbits, int32_t* __restrict__ first, int32_t* __restrict__ member_pos,
         float* __restrict__ member_w)
{
    extern __shared__ int lds[];   // cnt [BK_WAVES][ns] ints, then own [BK_WAVES][64 * IPT] 16-bit entry numbers
    __shared__ int wsum[BK_WAVES], wbelow[BK_WAVES];
    const int h = blockIdx.y, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int lo = blockIdx.x * S, ns = min(B, lo + S) - lo;   // this workgroup's slots [lo, lo + ns)
    if (ns <= 0) return;
    int* cnt = lds;
    unsigned short* own = reinterpret_cast<unsigned short*>(lds + BK_WAVES * ns) + wave * (64 * IPT);   // this wave's
    assign += (size_t)h * Le;
    evicted += (size_t)h * Le;
    sim += (size_t)h * Le;
    first += (size_t)h * (B + 1);
    member_pos += (size_t)h * Le;
    member_w += (size_t)h * Le;

    const int seg = wave * 64 * IPT;
    int a[IPT];
#pragma unroll
    for (int i = 0; i < IPT; ++i) a[i] = assign[min(seg + i * 64 + lane, Le - 1)];   // clamped: masked below
    for (int i = tid; i < BK_WAVES * ns; i += BK_THREADS) cnt[i] = 0;
    __syncthreads();
    int below_wave = 0, n_own = 0;
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const int e = seg + i * 64 + lane;
        int s = -1;
        if (e < Le) s = min(max(a[i], 0), B - 1) - lo;
        below_wave += __popcll(__ballot(e < Le && s < 0));
        const bool mine = s >= 0 && s < ns;
        const uint64_t mb = __ballot(mine);
        if (mine) {
            atomicAdd(&cnt[wave * ns + s], 1);
            own[n_own + mask_rank(mb)] = (unsigned short)(i * 64 + lane);
        }
        n_own += __popcll(mb);
    }
    // the wave's first two rows of own entries: their slot, position and cosine are fetched now and arrive while
    // the offsets are being worked out
    int pre_key[2], pre_pos[2];
    float pre_w[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const bool valid = u * 64 + lane < n_own;
        const int e = min(seg + (valid ? (int)own[u * 64 + lane] : 0), Le - 1);
        pre_key[u] = assign[e];
        pre_pos[u] = evicted[e];
        pre_w[u] = sim[e];
    }
    if (lane == 0) wbelow[wave] = below_wave;
    __syncthreads();

    const int per = (ns + BK_THREADS - 1) / BK_THREADS;
    const int a0 = min(ns, tid * per), a1 = min(ns, a0 + per);
    int local = 0;
    for (int s = a0; s < a1; ++s)
#pragma unroll
        for (int w = 0; w < BK_WAVES; ++w) local += cnt[w * ns + s];
    int incl = local;
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int run = incl - local;
#pragma unroll
    for (int w = 0; w < BK_WAVES; ++w) {
        run += wbelow[w] + ((w < wave) ? wsum[w] : 0);   // members of lower segments, then of lower slots
    }
    if (tid == 0 && lo + ns == B) first[B] = Le;
    for (int s = a0; s < a1; ++s) {
        first[lo + s] = run;
#pragma unroll
        for (int w = 0; w < BK_WAVES; ++w) {
            const int c = cnt[w * ns + s];
            cnt[w * ns + s] = run;
            run += c;
        }
    }
    __syncthreads();

    // one 64-entry row of the wave's list: rank lanes with equal slots, store, advance the slots' offsets
    auto place = [&](bool valid, int raw_slot, int pos, float sw) {
        const int key = valid ? min(max(raw_slot, 0), B - 1) - lo : 0;
        const uint64_t peers = match_key(key, valid, nbits);
        int base = 0;
        if (valid) {
            base = cnt[wave * ns + key];
            const int dst = base + mask_rank(peers);
            member_pos[dst] = pos;           // the set lists positions (ascending) and their cosines
            member_w[dst] = sw;
        }
        __builtin_amdgcn_wave_barrier();
        if (valid && (peers >> lane) == 1ull) cnt[wave * ns + key] = base + __popcll(peers);   // highest peer updates
        __builtin_amdgcn_wave_barrier();
    };
    if (n_own > 0) place(lane < n_own, pre_key[0], pre_pos[0], pre_w[0]);
    if (n_own > 64) place(64 + lane < n_own, pre_key[1], pre_pos[1], pre_w[1]);
    // further rows (a segment that most of the wave's entries belong to - few slots hold most members): each row's
    // slot, position and cosine are fetched while the row before it is being placed
    if (n_own > 128) {
        auto fetch_row = [&](int c0, int& key, int& pos, float& sw) {
            const bool valid = c0 + lane < n_own;
            const int e = min(seg + (valid ? (int)own[c0 + lane] : 0), Le - 1);
            key = assign[e];
            pos = evicted[e];
            sw = sim[e];
        };
        int key, pos;
        float sw;
        fetch_row(128, key, pos, sw);
        for (int c0 = 128; c0 < n_own; c0 += 64) {
            const int ck = key, cp = pos;
            const float cw = sw;
            if (c0 + 64 < n_own) fetch_row(c0 + 64, key, pos, sw);
            place(c0 + lane < n_own, ck, cp, cw);
        }
    }
}

// The merged row of a conserved token: its own row, its n members' weighted sum.
template <typename T>
__device__ __forceinline__ void merged_row(const raw8<T>& own, const float (&sum)[8], int n, int mode, T* __restrict__ out)
{
    float x[8];
    own.get(x);
    if (n > 0) {
        const float inv = 1.0f / (float)(n + 1);
        if (mode == LOOKM_MERGE_PIVOTAL)             // Eq. 11: (x_c + 1/2 sum (x_e + x_c)) / (n + 1)
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = (x[i] + 0.5f * fmaf((float)n, x[i], sum[i])) * inv;
        else                                         // Eq. 10 / Eq. 12: (x_c + sum w_e x_e) / (n + 1)
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = (x[i] + sum[i]) * inv;
    }
    store8(out, x);
}

// The members of the slots s0 .. s0 + ns - 1 by a workgroup of four waves, without a sort of the whole list: a wave goes through a
// quarter of the head's assignment list and keeps the entries of those slots, in order; then they are put into `members` by
// slot, the waves' shares in order.  begin[0 .. NG]: where each slot's members begin.  scratch_a: Le ints, scratch_b: 8 * NG ints.
constexpr int SCAN_MAX = 4096, SCAN_SLOTS = 32;      // entries of a list: 12 bits of a word, and 16 KB of them; slots: a lane each
__device__ __forceinline__ void collect_members(const int32_t* __restrict__ assign, int Le, int s0, int ns, int NG, int B, int* begin,
                                                float* scratch_a, float* scratch_b, unsigned short* members)
{
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    int* count = reinterpret_cast<int*>(scratch_b);                          // [wave][slot]
    int* next = count + 4 * NG + wave * NG;                                  // this wave's: where a slot's next member goes
    for (int i = tid; i < 4 * NG; i += 256) count[i] = 0;
    const int part = ((Le + 255) / 256) * 64, e_begin = min(Le, wave * part), e_end = min(Le, e_begin + part);
    uint32_t* own = reinterpret_cast<uint32_t*>(scratch_a) + e_begin;        // this wave's entries: slot << 12 | entry
    __syncthreads();
    int n = 0;
    for (int e0 = e_begin; e0 < e_end; e0 += 8 * 64) {                       // eight rows of 64 entries in flight
        int a[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) a[i] = assign[min(e0 + i * 64 + lane, Le - 1)];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int e = e0 + i * 64 + lane, key = min(max(a[i], 0), B - 1) - s0;
            const bool mine = e < e_end && key >= 0 && key < ns;
            const uint64_t m = __ballot(mine);
            if (mine) {
                own[n + mask_rank(m)] = (uint32_t)key << 12 | (uint32_t)e;
                atomicAdd(&count[wave * NG + key], 1);
            }
            n += __popcll(m);
        }
    }
    __syncthreads();
    int c[4], all = 0, before = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        c[w] = lane < NG ? count[w * NG + lane] : 0;
        before += w < wave ? c[w] : 0;
        all += c[w];
    }
    int incl = all;
#pragma unroll
    for (int off = 1; off < SCAN_SLOTS; off <<= 1) {
        const int v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
    }
    if (lane < NG) {
        next[lane] = incl - all + before;
        if (wave == 0) begin[lane] = incl - all;
        if (wave == 0 && lane == NG - 1) begin[NG] = incl;
    }
    __builtin_amdgcn_wave_barrier();
    for (int r0 = 0; r0 < n; r0 += 64) {
        const bool valid = r0 + lane < n;
        const uint32_t x = valid ? own[r0 + lane] : 0u;
        const int key = (int)(x >> 12);
        const uint64_t peers = match_key(key, valid, 5);
        int base = 0;
        if (valid) {
            base = next[key];
            members[base + mask_rank(peers)] = (unsigned short)(x & 4095u);
        }
        __builtin_amdgcn_wave_barrier();
        if (valid && (peers >> lane) == 1ull) next[key] = base + __popcll(peers);   // highest peer updates
        __builtin_amdgcn_wave_barrier();
    }
}

// G lanes per row, each lane 8 consecutive head dims of the key row and of the value row (both use the same set, the
// same weights and the same index reads).  A workgroup takes 256 / G consecutive slots, whose members are one stretch of the
// sorted lists, and its lane groups share out the MEMBERS evenly, whatever slots they belong to: set sizes are very uneven
// (half the slots have no member, some hundreds), and a lane group per slot spends as many memory latencies on the
// largest set of the chip as that has batches.  A group adds up its members in ascending order; where a slot ends inside
// its stretch the sum goes to LDS, a slot that several groups hold a part of is put together there in the order of
// the groups.  Members are fetched NB at a time (2 * NB row loads in flight per lane), their positions and weights a
// batch ahead; a short last batch repeats the last member and does not add it.  Bound by HBM: 32 heads x 12644, 2276
// conserved, 248 MB 53 -> 41 us; 40 x 5904, 3139 conserved 54 -> 39; 32 x 2896 18 -> 14, against a lane group per slot in the
// order of the set sizes, eight members of fp32 in flight (two workgroups a compute unit instead of four, and a plan of the
// slots by size to be made: sort 18.3 -> 16.3).  NB = 2: 43 us (12644) and 39.7 (5904), 6: 41.4 and 41.7, 8: 43.0 and 48.3.
// SCAN: the members come from the assignment list itself (collect_members), and member_pos and member_w are the evicted list and its
// cosines; otherwise first, member_pos and member_w are what k_bucket made.
template <typename T, int NB, bool SCAN>
__global__ void __launch_bounds__(256)
k_merge(const T* __restrict__ k, const T* __restrict__ v, const int32_t* __restrict__ kept, const int32_t* __restrict__ first,
        const int32_t* __restrict__ member_pos, const float* __restrict__ member_w, const int32_t* __restrict__ assign, int L, int d, int B,
        int Le, int mode, int lg_G, T* __restrict__ k_out, T* __restrict__ v_out)
{
    extern __shared__ unsigned short members[];                             // SCAN: entry numbers of the slots' members, slot by slot
    __shared__ int begin[257];                                              // of the slots' members; one more: the end
    __shared__ __attribute__((aligned(16))) float slot_sum[2][256 * 8];     // sums of slots that begin inside a group's stretch
    __shared__ __attribute__((aligned(16))) float head_sum[2][256 * 8];     // .. and of the end of one that began before
    // Heads vary fastest over the grid; the last eight blocks of slots come first, then the others in order.  Slots with many
    // members should not come last.  Those of the tokens that the scores picked lie anywhere, but the recent window is conserved
    // whatever its scores, and under the scores of an observation window its slots, the last ones, collect what resembles no
    // other (32 heads x 7613: half of a head's members in 64 of 2123 slots; merged last, four workgroups a head were at work by
    // themselves at the end: 45.7 -> 33.6 us; 32 x 2896 12.5 -> 11.6).
    const int blocks = (int)gridDim.y, tail = min(blocks >> 3, 8), y = (int)blockIdx.y, block = (y < tail) ? blocks - 1 - y : y - tail;
    const int h = blockIdx.x, tid = threadIdx.x, G = 1 << lg_G, NG = 256 >> lg_G, grp = tid >> lg_G, s0 = block * NG;
    const int c0 = (tid & (G - 1)) * 8, cc = (c0 < d) ? c0 : 0, slot = min(s0 + grp, B - 1);
    const int pos = kept[(size_t)h * B + slot];
    if (!SCAN)
        for (int i = tid; i <= NG; i += 256) begin[i] = (mode == LOOKM_MERGE_NONE) ? 0 : first[(size_t)h * (B + 1) + min(s0 + i, B)];
    k += (size_t)h * L * d + cc;
    v += (size_t)h * L * d + cc;
    // (SCAN: the lists first - behind the own rows, which wait for `pos`, they would come a round trip later.)
    if (SCAN) collect_members(assign + (size_t)h * Le, Le, s0, min(NG, B - s0), NG, B, begin, &slot_sum[0][0], &head_sum[0][0], members);
    raw8<T> own_k, own_v;
    own_k.load(k + (size_t)pos * d);
    own_v.load(v + (size_t)pos * d);
    __syncthreads();
    const int m0 = begin[0], M = begin[NG] - m0, per = (M + NG - 1) >> (8 - lg_G);      // members of a group
    const int t_end = min(m0 + (grp + 1) * per, m0 + M);
    int t = m0 + grp * per;
    if (t < t_end) {
        member_pos += (size_t)h * Le;
        member_w += (size_t)h * Le;
        const bool weighted = (mode == LOOKM_MERGE_WEIGHTED);
        int c = 0;                                                          // the slot that member t belongs to
        for (int step = NG >> 1; step > 0; step >>= 1) c += (begin[c + step] <= t) ? step : 0;
        bool head = begin[c] < t;
        int c_end = begin[c + 1];
        float ak[8], av[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) ak[i] = av[i] = 0.f;
        auto flush = [&]() {
            float* to_k = head ? &head_sum[0][tid * 8] : &slot_sum[0][((c << lg_G) + (tid & (G - 1))) * 8];
            float* to_v = to_k + 256 * 8;
            store8(to_k, ak);
            store8(to_v, av);
            head = false;
#pragma unroll
            for (int i = 0; i < 8; ++i) ak[i] = av[i] = 0.f;
        };
        int p[NB];
        float w[NB];
        auto fetch_members = [&](int from) {
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const int tt = min(from + j, t_end - 1), e = SCAN ? members[tt] : tt;
                p[j] = member_pos[e];
                w[j] = weighted ? member_w[e] : 1.0f;
            }
        };
        fetch_members(t);
        for (; t < t_end; t += NB) {
            raw8<T> xk[NB], xv[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                xk[j].load(k + (size_t)p[j] * d);
                xv[j].load(v + (size_t)p[j] * d);
            }
            float wc[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) wc[j] = w[j];
            if (t + NB < t_end) fetch_members(t + NB);
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                if (t + j < t_end) {
                    if (t + j == c_end) {
                        flush();
                        do { c_end = begin[++c + 1]; } while (c_end <= t + j);          // (slots without members)
                    }
                    float e[8];
                    xk[j].get(e);
#pragma unroll
                    for (int i = 0; i < 8; ++i) ak[i] = fmaf(e[i], wc[j], ak[i]);
                    xv[j].get(e);
#pragma unroll
                    for (int i = 0; i < 8; ++i) av[i] = fmaf(e[i], wc[j], av[i]);
                }
            }
        }
        flush();
    }
    __syncthreads();
    if (s0 + grp >= B || c0 >= d) return;
    const int n = begin[grp + 1] - begin[grp];       // L_sim: size of this slot's similarity set
    float sk[8], sv[8];
    if (n > 0) {
        load8(&slot_sum[0][tid * 8], sk);
        load8(&slot_sum[1][tid * 8], sv);
        const int g_first = (begin[grp] - m0) / per, g_last = (begin[grp + 1] - 1 - m0) / per;
        for (int g = g_first + 1; g <= g_last; ++g) {
            float e[8];
            load8(&head_sum[0][((g << lg_G) + (tid & (G - 1))) * 8], e);
#pragma unroll
            for (int i = 0; i < 8; ++i) sk[i] += e[i];
            load8(&head_sum[1][((g << lg_G) + (tid & (G - 1))) * 8], e);
#pragma unroll
            for (int i = 0; i < 8; ++i) sv[i] += e[i];
        }
    }
    const size_t out_off = ((size_t)h * B + slot) * d + c0;
    merged_row(own_k, sk, n, mode, k_out + out_off);
    merged_row(own_v, sv, n, mode, v_out + out_off);
}

// The same for the shortest lists: a wave looks after 64 / G consecutive slots, loads the head's whole assignment list by
// itself and puts the few entries of its slots, in order, into LDS.  All of it is a chain of
// memory latencies; this one is a kernel and a round trip shorter (2 heads x 256 x 64 fp32, the whole layer: 27.0 -> 23.4 us; 23.8 when
// a wave read positions and cosines of its own entries after it had found them).
// Members are added up by the slot's lane group, up to SHARED of them: one after the other they would make the largest set the
// time of the kernel.  (8 heads, 256 members on 256 slots x 128 bf16, us, a slot's own lane group for all / shared / the merge whose
// workgroups scan / sort and merge: all in one set 41.9 / 13.5 / 9.6 / 13.5, half of them 24.2 / 11.1 / 8.7 / 12.1, even sets 5.1 / 5.2 /
// 5.6 / 8.4; 2 heads, 256 on 154 x 64 fp32 34.0 / 7.7 / 9.2 / 13.1, 20.9 / 7.9 / 8.9 / 12.2, 4.8 / 4.9 / 5.4 / 8.0.)
constexpr int DIRECT_MAX = 256, SHARED = 32;
template <typename T, int NB>
__global__ void __launch_bounds__(256)
k_merge_direct(const T* __restrict__ k, const T* __restrict__ v, const int32_t* __restrict__ kept, const int32_t* __restrict__ evicted,
               const int32_t* __restrict__ assign, const float* __restrict__ sim, int L, int d, int B, int Le, int mode, int G,
               T* __restrict__ k_out, T* __restrict__ v_out)
{
    constexpr int ROWS = DIRECT_MAX / 64;
    __shared__ int member_pos[4][DIRECT_MAX];           // the wave's members, slot by slot
    __shared__ float member_w[4][DIRECT_MAX];
    __shared__ int first[4][9], next[4][8];             // of each slot: its first member, and where the next one goes
    const int h = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int slots = 64 / G, s0 = ((int)blockIdx.y * 4 + wave) * slots, g = lane / G, c0 = lane % G * 8;
    assign += (size_t)h * Le;
    evicted += (size_t)h * Le;
    sim += (size_t)h * Le;
    const int slot = min(s0 + g, B - 1), pos = kept[(size_t)h * B + slot];
    // the whole list at once, positions and cosines too: what belongs to other waves is cheaper than a round trip more for the own
    int key[ROWS], p[ROWS];
    float w[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        const int e = min(i * 64 + lane, Le - 1);
        key[i] = assign[e];
        p[i] = evicted[e];
        w[i] = sim[e];
    }
    if (lane < 8) next[wave][lane] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        key[i] = i * 64 + lane < Le ? min(max(key[i], 0), B - 1) - s0 : -1;
        if (key[i] >= 0 && key[i] < slots) atomicAdd(&next[wave][key[i]], 1);
        else key[i] = -1;
    }
    __syncthreads();
    if (lane < 9) {
        int before = 0;
        for (int i = 0; i < min(lane, 8); ++i) before += next[wave][i];
        first[wave][lane] = before;
    }
    __syncthreads();
    if (lane < 8) next[wave][lane] = first[wave][lane];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        if (!__any(key[i] >= 0)) continue;
        const bool valid = key[i] >= 0;
        const uint64_t peers = match_key(key[i], valid, 3);
        int base = 0;
        if (valid) {
            base = next[wave][key[i]];
            member_pos[wave][base + mask_rank(peers)] = p[i];
            member_w[wave][base + mask_rank(peers)] = w[i];
        }
        __builtin_amdgcn_wave_barrier();
        if (valid && (peers >> lane) == 1ull) next[wave][key[i]] = base + __popcll(peers);   // highest peer updates
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    const int cc = (c0 < d) ? c0 : 0;
    k += (size_t)h * L * d + cc;
    v += (size_t)h * L * d + cc;
    raw8<T> own_k, own_v;
    own_k.load(k + (size_t)pos * d);
    own_v.load(v + (size_t)pos * d);
    float sk[8], sv[8];
    auto add_up = [&](int t, int t_end) {               // ascending position; a short last batch repeats the last member
#pragma unroll
        for (int i = 0; i < 8; ++i) sk[i] = sv[i] = 0.f;
        for (; t < t_end; t += NB) {
            raw8<T> xk[NB], xv[NB];
            float w[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const int tt = min(t + j, t_end - 1), p = member_pos[wave][tt];
                xk[j].load(k + (size_t)p * d);
                xv[j].load(v + (size_t)p * d);
                w[j] = (mode == LOOKM_MERGE_WEIGHTED) ? member_w[wave][tt] : 1.0f;
            }
#pragma unroll
            for (int j = 0; j < NB; ++j)
                if (t + j < t_end) {
                    float e[8];
                    xk[j].get(e);
#pragma unroll
                    for (int i = 0; i < 8; ++i) sk[i] = fmaf(e[i], w[j], sk[i]);
                    xv[j].get(e);
#pragma unroll
                    for (int i = 0; i < 8; ++i) sv[i] = fmaf(e[i], w[j], sv[i]);
                }
        }
    };
    const int n = first[wave][g + 1] - first[wave][g];
    const size_t out_off = ((size_t)h * B + slot) * d + c0;
    const bool writes = s0 + g < B && c0 < d;
    // A set of more than SHARED members is added up by all the wave's lane groups, a stretch by each.
    for (uint64_t large = __ballot(n > SHARED); large != 0;) {
        const int at = __builtin_ctzll(large) / G, t0 = first[wave][at], t1 = first[wave][at + 1], per = (t1 - t0 + slots - 1) / slots;
        large &= ~0ull << at * G << (G - 1) << 1;
        add_up(t0 + g * per, min(t0 + g * per + per, t1));
        for (int step = G; step < 64; step <<= 1)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                sk[i] += __shfl_xor(sk[i], step);
                sv[i] += __shfl_xor(sv[i], step);
            }
        if (g == at && writes) {
            merged_row(own_k, sk, n, mode, k_out + out_off);
            merged_row(own_v, sv, n, mode, v_out + out_off);
        }
    }
    if (n > SHARED || !writes) return;
    add_up(first[wave][g], first[wave][g + 1]);
    merged_row(own_k, sk, n, mode, k_out + out_off);
    merged_row(own_v, sv, n, mode, v_out + out_off);
}

}  // namespace lookm

namespace lookm_host {

// Segments per head: as many as make no more workgroups than there are compute units (40 heads x 2765 entries in seven segments,
// 280 workgroups, 8.0 us, in six 6.7; whole layers of 24, 40, 64, 96, 128, 160, 200 and 255 heads with one segment more: the same
// within 0.4 %), and no more than BK_MAX_SEG slots in one segment.
static void bucket_segments(int H, int B, int& S, int& NS)
{
    int ns = std::max(1, 256 / H);
    if (ns > 16) ns = 16;
    const int need = (B + lookm::BK_MAX_SEG - 1) / lookm::BK_MAX_SEG;
    if (ns < need) ns = need;
    if (ns > B) ns = B;
    S = (B + ns - 1) / ns;
    NS = (B + S - 1) / S;
}

// log2 of the lanes per row
static int merge_lanes(int d)
{
    int lg = 0;
    while ((8 << lg) < d) ++lg;
    return lg;
}

template <typename T>
static void launch_merge_t(const T* k, const T* v, const int32_t* kept, const int32_t* first, const int32_t* member_pos,
                           const float* member_w, const int32_t* assign, int H, int L, int d, int B, int mode, T* k_out, T* v_out, hipStream_t st)
{
    const int lg_G = merge_lanes(d), slots = 256 >> lg_G;
    const dim3 grid(H, (B + slots - 1) / slots);
    if (assign != nullptr)
        hipLaunchKernelGGL((lookm::k_merge<T, 4, true>), grid, dim3(256), (L - B) * sizeof(unsigned short), st, k, v, kept, first, member_pos,
                           member_w, assign, L, d, B, L - B, mode, lg_G, k_out, v_out);
    else
        hipLaunchKernelGGL((lookm::k_merge<T, 4, false>), grid, dim3(256), 0, st, k, v, kept, first, member_pos, member_w, assign, L, d, B,
                           L - B, mode, lg_G, k_out, v_out);
}

template <int IPT>
static int launch_bucket(const int32_t* assign, const int32_t* evicted, const float* sim, int H, int Le, int B, int S, int NS,
                         int32_t* first, int32_t* member_pos, float* member_w, hipStream_t st)
{
    const size_t lds = (size_t)lookm::BK_WAVES * (S * sizeof(int) + 64 * IPT * sizeof(unsigned short));
    int nbits = 1;
    while ((1 << nbits) < S) ++nbits;
    hipLaunchKernelGGL(lookm::k_bucket<IPT>, dim3(NS, H), dim3(lookm::BK_THREADS), lds, st, assign, evicted, sim,
                       Le, B, S, nbits, first, member_pos, member_w);
    return LOOKM_OK;
}

int launch_merge(const void* k, const void* v, const int32_t* kept, const int32_t* evicted, const int32_t* assign,
                 const float* sim, int H, int L, int d, lookm_dtype dt, int budget, int mode, int32_t* first,
                 int32_t* member_pos, float* member_w, void* k_out, void* v_out, hipStream_t st)
{
    const int B = budget, Le = L - B;
    if (B == 0) return LOOKM_OK;
    const LaunchCheck check;
    if (Le == 0) mode = LOOKM_MERGE_NONE;
    const int G = 1 << merge_lanes(d);
    // The shortest lists: a wave collects the members of its slots by itself.  The merge alone, even sets, us, this way / by the merge whose
    // workgroups scan (below) / sorted: 2 heads, 102 entries in 154 slots x 64 fp32 4.6 / 5.0 / 7.7; 8, 128 in 143 x 128 fp32 4.7 / 5.3 /
    // 8.0; 8, 256 in 64 x 128 bf16 5.9 / 6.6 / 9.4; 32, 256 in 64 x 64 bf16 6.0 / 6.8 / 9.6.  Whole layers beyond 256 entries, this way in
    // two and four times the registers / scan: 1 head, 346 in 386 x 80 28.3 / 27.8; 2, 500 in 200 x 64 fp32 34.2 / 33.1; 8, 500 in 200 x 128
    // 46.5 / 45.3.  A lane group has eight lanes and more, so that a wave has at most eight slots.
    if (mode != LOOKM_MERGE_NONE && Le <= lookm::DIRECT_MAX && Le <= 4 * (long)B && G >= 8 && (size_t)H * B * G / 64 <= 2048) {
        const int spb = 4 * (64 / G);
        auto go = [&](auto type) {
            typedef decltype(type) T;
            hipLaunchKernelGGL((lookm::k_merge_direct<T, 8>), dim3(H, (B + spb - 1) / spb), dim3(256), 0, st, (const T*)k, (const T*)v, kept,
                               evicted, assign, sim, L, d, B, Le, mode, G, (T*)k_out, (T*)v_out);
        };
        if (dt == LOOKM_BF16) go(lookm::bf16_t{});
        else go(float{});
        mark(LOOKM_K_MERGE);
        return check.status();
    }
    // Short lists: every workgroup of the merge goes through the head's list, instead of a kernel that sorts it.  That kernel and
    // its launch are 6 to 8 us whatever the merge's size (a little less for the shortest lists); going through the list is a
    // round trip and five barriers for every round of workgroups, four to a compute unit: the line is a number of workgroups.  Whole layers, us, sort and
    // merge / scan: 32 heads x 128 bf16, 300 entries, 2560 workgroups 88.0 / 85.4, 3584 104.6 / 103.5, 5120 134.8 / 134.8, 6144 151.3 / 153.0,
    // 8192 209 / 211; 60 entries, 2560 70.4 / 69.8, 3072 81.9 / 81.4, 4096 92.6 / 93.2, 8192 179 / 181; 128 heads, 700 entries, 5120 169.6
    // / 168.6, 8192 204.3 / 205.3; 32 heads x 256, 300 entries, 5120 138.4 / 138.2, 8192 218.5 / 223.0; 32 x 128 fp32, 300, 5120 524 / 520;
    // 240 entries, 3136 91.9 / 90.5, 180, 3584 62.1 / 61.0; rows that leave lanes idle, 32 x 80, 461, 3232 92.8 / 91.5, 691, 3936 87.2 / 88.4, 4880 128.4 / 130.6.
    // Entries times workgroups: past 2048 entries a second round trip; one stream gains up to 2 us more of it (32 x 84 workgroups
    // x 2765 226.4 / 223.9), but two streams, one job's sort beside the other's long kernels, lose: a batch of 32 x 84 x 2733 6 us a layer.
    const long workgroups = (long)H * ((B + (256 / G) - 1) / (256 / G));
    const bool scan = mode != LOOKM_MERGE_NONE && G >= 8 && Le <= lookm::SCAN_MAX && workgroups <= (8 * G != d || Le < 256 ? 3584 : 5120) &&
                      workgroups * Le <= 4l << 20;
    static_assert(256 / 8 <= lookm::SCAN_SLOTS, "a lane for each slot of a workgroup");
    if (scan) {
        member_pos = const_cast<int32_t*>(evicted);          // (read only) by entry number
        member_w = const_cast<float*>(sim);
    } else if (mode != LOOKM_MERGE_NONE) {
        int S, NS;
        bucket_segments(H, B, S, NS);
        const int per_thread = (Le + lookm::BK_THREADS - 1) / lookm::BK_THREADS;
        int rc;
        if (per_thread <= 4)
            rc = launch_bucket<4>(assign, evicted, sim, H, Le, B, S, NS, first, member_pos, member_w, st);
        else if (per_thread <= 8)
            rc = launch_bucket<8>(assign, evicted, sim, H, Le, B, S, NS, first, member_pos, member_w, st);
        else if (per_thread <= 16)
            rc = launch_bucket<16>(assign, evicted, sim, H, Le, B, S, NS, first, member_pos, member_w, st);
        else if (per_thread <= 32)
            rc = launch_bucket<32>(assign, evicted, sim, H, Le, B, S, NS, first, member_pos, member_w, st);
        else
            return LOOKM_ERR_UNSUPPORTED;
        if (rc != LOOKM_OK) return rc;
        mark(LOOKM_K_BUCKET);
    }
    if (dt == LOOKM_BF16)
        launch_merge_t((const lookm::bf16_t*)k, (const lookm::bf16_t*)v, kept, first, member_pos, member_w, scan ? assign : nullptr, H, L, d,
                       B, mode, (lookm::bf16_t*)k_out, (lookm::bf16_t*)v_out, st);
    else
        launch_merge_t((const float*)k, (const float*)v, kept, first, member_pos, member_w, scan ? assign : nullptr, H, L, d, B, mode,
                       (float*)k_out, (float*)v_out, st);
    mark(LOOKM_K_MERGE);
    return check.status();
}

template <int IPT> static bool bucket_attribute()
{
    return hipFuncSetAttribute((const void*)lookm::k_bucket<IPT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               lookm::BK_WAVES * (lookm::BK_MAX_SEG * 4 + 64 * IPT * 2)) == hipSuccess;
}

int set_attributes_merge()
{
    return (bucket_attribute<4>() && bucket_attribute<8>() && bucket_attribute<16>() && bucket_attribute<32>())
               ? LOOKM_OK : LOOKM_ERR_DEVICE;
}

}  // namespace lookm_host
