// Attention of one new token over a cache (Section 3.1, Eq. 3): out = Softmax(q K^T / sqrt(d)) V, per head,
// over the first S rows of a [H, rows, d] cache - the step that the compressed cache of Eq. 6-7 exists for.
// Bound by HBM: every key row and every value row in use is read exactly once.
//
// The cache rows of a head are cut into `nsplit` contiguous pieces, one workgroup each, so that a few heads fill the
// chip.  Inside a workgroup G = d/8 (rounded up to a power of two) lanes share a row, eight elements per lane; the
// workgroup takes a step of 4 * 256 / G rows at a time (four key loads and four value loads in flight per lane), and every
// lane group keeps a running (max, sum, weighted value) in base 2 with the softmax scale folded in.  The groups of a
// workgroup, and then the pieces of a head, are merged in a fixed order, so the result is bitwise repeatable.
// Measured over caches that don't stay on the chip, both kernels: 32 heads x 5000 rows of bf16 (82 MB) 37.0 -> 21.0 us,
// x 12644 (207 MB) 64 -> 40.5 us = 5.1 TB/s; fp32 x 12644 (414 MB) 81 -> 74 us.  What the first version lost: row chunks
// converted to fp32 as they arrived (104 registers, half the workgroups in flight), sums across lanes through LDS
// permutes, four adjacent rows per lane group (a wave's load spread over sixteen rows), a merge with three barriers.
#include "common.h"

#include <algorithm>
#include <mutex>

namespace lookm {

constexpr int DC_THREADS = 256;
constexpr int DC_ROWS = 4;          // rows per lane group and step (the NaN test below adds four by name)
constexpr int DC_MAX_SPLIT = 256;
constexpr int DC_DIMS = 32;         // output dims per workgroup of the merge

// sum over the G lanes of a group (groups aligned to G lanes).  Up to sixteen lanes by data-parallel moves of the vector
// ALU: exchanges of neighbours and pairs, then mirrors of half rows and rows, which are exchanges too once the lanes that
// trade places hold equal sums.
template <int CTRL> __device__ __forceinline__ float dpp_add(float x)
{
    return x + __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xf, 0xf, true));
}
template <int G> __device__ __forceinline__ float group_sum(float x)
{
    if (G >= 2) x = dpp_add<0xB1>(x);     // quad_perm 1 0 3 2
    if (G >= 4) x = dpp_add<0x4E>(x);     // quad_perm 2 3 0 1
    if (G >= 8) x = dpp_add<0x141>(x);    // row_half_mirror
    if (G >= 16) x = dpp_add<0x140>(x);   // row_mirror
    if (G >= 32) x += __shfl_xor(x, 16);
    return x;
}

// Partial results of a call: weighted value sums [H][nsplit][d], then (running max in base 2, sum of weights) [H][nsplit].
template <typename T, int G>
__global__ void __launch_bounds__(DC_THREADS)
k_decode_partial(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, int rows, int S, int d,
                 int nsplit, float scale2, float* __restrict__ part, float2* __restrict__ part_ml)
{
    constexpr int NG = DC_THREADS / G, W8 = G * 8;
    __shared__ __attribute__((aligned(16))) float gv[NG * W8];
    __shared__ float gm[NG], gl[NG];
    const int h = blockIdx.y, piece = blockIdx.x, tid = threadIdx.x;
    const int grp = tid / G, c0 = (tid % G) * 8;
    const bool live = c0 < d;       // lanes past the head dim (d not a power of two times 8) carry zeros
    const int per = (S + nsplit - 1) / nsplit;
    const int r_begin = piece * per, r_end = min(S, r_begin + per);
    const int cc = live ? c0 : 0;
    k += (size_t)h * rows * d + cc;
    v += (size_t)h * rows * d + cc;

    raw8<T> qr;
    qr.load(q + (size_t)h * d + cc);
    float qv[8];
    float m = -INFINITY, l = 0.f, o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int r0 = r_begin; r0 < r_end; r0 += NG * DC_ROWS) {
        raw8<T> kr[DC_ROWS], vr[DC_ROWS];
#pragma unroll
        for (int j = 0; j < DC_ROWS; ++j)                  // a short last step re-reads the last row with weight 0
            kr[j].load(k + (size_t)min(r0 + j * NG + grp, r_end - 1) * d);
#pragma unroll
        for (int j = 0; j < DC_ROWS; ++j) vr[j].load(v + (size_t)min(r0 + j * NG + grp, r_end - 1) * d);
        qr.get(qv);
        float s[DC_ROWS];
#pragma unroll
        for (int j = 0; j < DC_ROWS; ++j) {
            float x[8], dot = 0.f;
            kr[j].get(x);
#pragma unroll
            for (int i = 0; i < 8; ++i) dot = fmaf(qv[i], x[i], dot);
            s[j] = live ? dot : 0.f;
        }
#pragma unroll
        for (int j = 0; j < DC_ROWS; ++j) s[j] = (r0 + j * NG + grp < r_end) ? group_sum<G>(s[j]) * scale2 : -INFINITY;
        float mn = m;
#pragma unroll
        for (int j = 0; j < DC_ROWS; ++j) mn = fmaxf(mn, s[j]);
        // a group without a row yet, or whose logits are all -inf: everything stays zero.  (fmaxf passes a NaN over; the sum
        // does not, and a row whose logit is NaN has to reach the result.)
        if (mn != -INFINITY || (s[0] + s[1]) + (s[2] + s[3]) != -INFINITY) {
            const float keep = __builtin_amdgcn_exp2f(m - mn);
            l *= keep;
#pragma unroll
            for (int i = 0; i < 8; ++i) o[i] *= keep;
#pragma unroll
            for (int j = 0; j < DC_ROWS; ++j)
                if (r0 + j * NG + grp < r_end) {           // (a row read again may hold an infinity: 0 would not undo it)
                    float x[8];
                    vr[j].get(x);
                    const float p = __builtin_amdgcn_exp2f(s[j] - mn);
                    l += p;
#pragma unroll
                    for (int i = 0; i < 8; ++i) o[i] = fmaf(p, x[i], o[i]);
                }
            m = mn;
        }
    }

    // merge the lane groups of the workgroup, group 0 first: every dim's thread works out the groups' weights for itself
    if (tid % G == 0) { gm[grp] = m; gl[grp] = l; }
    *reinterpret_cast<float4*>(&gv[grp * W8 + c0]) = make_float4(o[0], o[1], o[2], o[3]);
    *reinterpret_cast<float4*>(&gv[grp * W8 + c0 + 4]) = make_float4(o[4], o[5], o[6], o[7]);
    __syncthreads();
    if (tid >= d) return;
    float M = -INFINITY, acc = 0.f, sum = 0.f;
#pragma unroll 16
    for (int g = 0; g < NG; ++g) M = fmaxf(M, gm[g]);
#pragma unroll 16
    for (int g = 0; g < NG; ++g) {
        const float w = (gm[g] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(gm[g] - M);
        acc = fmaf(gv[g * W8 + tid], w, acc);
        sum = fmaf(gl[g], w, sum);
    }
    const size_t at = (size_t)h * nsplit + piece;
    part[at * d + tid] = acc;
    if (tid == 0) part_ml[at] = make_float2(M, sum);
}

// Merges the pieces of a head and normalises, DC_DIMS output dims per workgroup.  Every wave works out the pieces' weights
// 2^(max - M) and the denominator for itself (four pieces per lane, no barrier); thread (slice, c) sums dim c over the
// pieces slice, slice + 8, ..., its first loads in flight together with those of the maxima, and the slices are added in
// order.
template <typename T>
__global__ void __launch_bounds__(DC_THREADS)
k_decode_merge(const float* __restrict__ part, const float2* __restrict__ part_ml, int d, int nsplit, T* __restrict__ out)
{
    constexpr int NSL = DC_THREADS / DC_DIMS, PER = DC_MAX_SPLIT / 64, AHEAD = 8;
    __shared__ float wgt[DC_THREADS / 64][DC_MAX_SPLIT];
    __shared__ float red[NSL][DC_DIMS];
    const int h = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int slice = tid / DC_DIMS, c = blockIdx.y * DC_DIMS + tid % DC_DIMS;
    const float* p = part + (size_t)h * nsplit * d + min(c, d - 1);
    const float2* ml = part_ml + (size_t)h * nsplit;
    float2 x[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        x[i] = ml[min(i * 64 + lane, nsplit - 1)];
        if (i * 64 + lane >= nsplit) x[i] = make_float2(-INFINITY, 0.f);
    }
    float a[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) a[i] = p[(size_t)min(slice + i * NSL, nsplit - 1) * d];
    float M = -INFINITY;
#pragma unroll
    for (int i = 0; i < PER; ++i) M = fmaxf(M, x[i].x);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) M = fmaxf(M, __shfl_xor(M, off));
    float den = 0.f;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const float w = (x[i].x == -INFINITY) ? 0.f : exp2f(x[i].x - M);     // an empty piece: weight 0
        wgt[wave][i * 64 + lane] = w;
        den = fmaf(x[i].y, w, den);
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) den += __shfl_xor(den, off);
    __builtin_amdgcn_wave_barrier();
    const float* weight = wgt[wave] + unknown_zero();                       // the wave reads what its own lanes wrote
    float num = 0.f;
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
        if (slice + i * NSL < nsplit) num = fmaf(a[i], weight[slice + i * NSL], num);
#pragma unroll 8
    for (int s = slice + AHEAD * NSL; s < nsplit; s += NSL) num = fmaf(p[(size_t)s * d], weight[s], num);
    red[slice][tid % DC_DIMS] = num;
    __syncthreads();
    if (slice == 0 && c < d) {
        float tot = 0.f;
#pragma unroll
        for (int sl = 0; sl < NSL; ++sl) tot += red[sl][tid];
        elem<T>::store(out + (size_t)h * d + c, tot / den);
    }
}

}  // namespace lookm

namespace lookm_host {

// rows a workgroup of the partial kernel covers in one step
static int decode_step_rows(int d)
{
    int G = 1;
    while (G * 8 < d) G <<= 1;
    return lookm::DC_THREADS / G * lookm::DC_ROWS;
}

// Pieces per head: one per step while that makes at most 1536 workgroups - what the chip holds at once, six to a compute
// unit - and as few steps more per piece as it takes beyond that.  Between one and four steps nothing differs by more than
// 5 % (32 heads x 2311: 12.2, 13.0, 12.5, 13.3 us; x 5000: 20.4, 21.1, 20.6, 21.3), at six the short caches run out of
// workgroups (15.1 us), and every piece more is a row of partial results for the merge.
static int decode_pieces(int H, int S, int d)
{
    const int step = decode_step_rows(d), steps = (S + step - 1) / step;
    const long k = std::max<long>(1, ((long)H * steps + 1535) / 1536);
    const int n = (int)((steps + k - 1) / k);
    return std::min(n, lookm::DC_MAX_SPLIT);
}

size_t decode_scratch_bytes(int H, int d) { return (size_t)H * lookm::DC_MAX_SPLIT * (d + 2) * sizeof(float); }

// upper bound of the bytes of partial results one call writes and reads (at most decode_scratch_bytes), and what the entry
// point without a workspace refuses by: one piece per step, or per two steps from 1024 such pieces on
size_t decode_partial_bytes(int H, int S, int d)
{
    const int step = decode_step_rows(d);
    int n = (S + step - 1) / step;
    if ((long)H * (n / 2) >= 1024) n = (n + 1) / 2;
    return (size_t)H * std::min(n, lookm::DC_MAX_SPLIT) * (d + 2) * sizeof(float);
}

template <typename T>
static int launch_decode_t(const T* q, const T* k, const T* v, int H, int rows, int S, int d, T* out, float* part,
                           hipStream_t st)
{
    const LaunchCheck check;
    const int nsplit = decode_pieces(H, S, d);
    const float scale2 = lookm::kLog2e / sqrtf((float)d);
    const size_t values = (size_t)H * nsplit * d;          // d is a multiple of 8: what follows is aligned
    float2* ml = reinterpret_cast<float2*>(part + values);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nsplit, H), dim3(lookm::DC_THREADS), 0, st, q, k, v, rows, S, d, nsplit, scale2, part, ml);
    };
    if (d <= 8) go(lookm::k_decode_partial<T, 1>);
    else if (d <= 16) go(lookm::k_decode_partial<T, 2>);
    else if (d <= 32) go(lookm::k_decode_partial<T, 4>);
    else if (d <= 64) go(lookm::k_decode_partial<T, 8>);
    else if (d <= 128) go(lookm::k_decode_partial<T, 16>);
    else go(lookm::k_decode_partial<T, 32>);
    hipLaunchKernelGGL(lookm::k_decode_merge<T>, dim3(H, (d + lookm::DC_DIMS - 1) / lookm::DC_DIMS), dim3(lookm::DC_THREADS), 0, st, part,
                       ml, d, nsplit, out);
    return check.status();
}

int launch_decode(const void* q, const void* k, const void* v, int H, int rows, int S, int d, lookm_dtype dt, void* out,
                  float* part, hipStream_t st)
{
    if (dt == LOOKM_BF16)
        return launch_decode_t((const lookm::bf16_t*)q, (const lookm::bf16_t*)k, (const lookm::bf16_t*)v, H, rows, S, d,
                               (lookm::bf16_t*)out, part, st);
    return launch_decode_t((const float*)q, (const float*)k, (const float*)v, H, rows, S, d, (float*)out, part, st);
}

// ---- scratch for callers that may not allocate ---------------------------------------------------------------
// lookm_decode_attention_noalloc keeps the partial results of its two kernels in this array instead of a
// caller's workspace.  Every GPU the library runs on holds its own copy, at its own address, until the process
// ends.  In host code the array's name is only a stand-in for the symbol: the device address is asked for once per
// device (with that device current) and kept; kernels get that pointer as their argument, exactly as they get the
// caller's workspace in lookm_decode_attention.  Nothing in the array has to start at zero: the first kernel writes
// every partial the second one reads.
static __device__ __align__(256) unsigned char scratch[LOOKM_DECODE_NOALLOC_SCRATCH_BYTES];

static std::mutex g_scratch_mutex;
static float* g_scratch_ptr[64];     // per device; null until resolved

int decode_static_scratch_setup()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return LOOKM_ERR_DEVICE;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] != nullptr) return LOOKM_OK;
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return LOOKM_ERR_DEVICE;
    g_scratch_ptr[dev] = static_cast<float*>(ptr);
    return LOOKM_OK;
}

// the current device's copy of the array, or null when decode_static_scratch_setup has not succeeded on it
float* decode_static_scratch()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    return g_scratch_ptr[dev];
}

}  // namespace lookm_host
