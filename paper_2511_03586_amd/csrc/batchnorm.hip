// Batch normalisation with batch statistics for gfx950 ("batchnorm" rows of the operator
// table, Section 4.3 of the paper; its MI300A case study is this operator: the statistics
// are computed first, then a streaming kernel normalises).  x is NCHW; a channel's data are
// N planes of H*W contiguous elements.
//
//  * bn_partial_kernel: a workgroup reduces one segment (<= 16384 elements) of a channel, held in registers:
//    part of a plane, or several whole planes where they are small; provisional mean, then first and second
//    moments of the shifted data (the corrected two-pass form of the LayerNorm kernel), written as
//    (mean_hi, mean_lo, M2).
//  * bn_channel_kernel: channels that a workgroup holds in registers, in one launch.
//  * bn_apply_kernel: streaming y = (x - mean) * scale + beta, 16-byte accesses, on the same segments.  The channel's
//    segments are merged in double precision, by every workgroup while its loads fly if there are at most
//    256 of them, else by bn_finalize_kernel (one workgroup per channel).
// Planes of any size and alignment use 16-byte loads (row_io.h: the chunk that would overhang a plane starts
// early and its shared elements count once).
// The partials live in a caller-supplied workspace (perf_batchnorm_workspace_bytes): no
// atomics, results bit-identical from run to run.
#include <atomic>
#include <type_traits>
#include "row_io.h"
#include "host_utils.h"

namespace perf {

constexpr int kBnSeg = 16384;  // elements per segment: 256 threads x 64

__device__ __forceinline__ float bn_block_sum(float v, float *red)
{
    v = wave_allreduce(v, OpSum{});
    __syncthreads();  // red may still be read from the previous use
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

constexpr int kBnFuseSegs = 256;  // segments per channel up to which the apply kernel merges them itself

// How a channel is cut.  Planes of more than half a segment are split (spp segments each); smaller ones are grouped,
// G to a segment.  An item is a chunk of 16 bytes of x; a segment's items are numbered through its planes.
struct BnGeom {
    int64_t HW;
    int C, N;
    int64_t cpp;   // chunks per plane
    int G, spp;    // planes per segment (0: split), segments per plane when split
    int segs;      // segments per channel
    uint32_t m_cpp;
    __device__ __forceinline__ int64_t count(int s) const  // elements of segment s
    {
        return G ? (int64_t)min(G, N - s * G) * HW : min((int64_t)kBnSeg, HW - (int64_t)(s % spp) * kBnSeg);
    }
};

template <typename T, int NJ, bool RAG, int THREADS = 256>
struct BnItems {  // this thread's items of a segment
    static constexpr int E = Elem<T>::kPerChunk;
    const BnGeom &g;
    int64_t base, c0;  // first element of the segment's first plane (channel c); first chunk when split
    int total;         // items of the segment
    __device__ __forceinline__ BnItems(const BnGeom &g_, int c, int s) : g(g_)
    {
        const int n0 = g.G ? s * g.G : s / g.spp, part = g.G ? 0 : s % g.spp;
        base = ((int64_t)n0 * g.C + c) * g.HW;
        c0 = (int64_t)part * (kBnSeg / E);
        total = g.G ? min(g.G, g.N - n0) * (int)g.cpp : (int)min((int64_t)(kBnSeg / E), g.cpp - c0);
    }
    __device__ __forceinline__ bool all() const { return total == NJ * THREADS; }
    __device__ __forceinline__ bool valid(int j) const { return j * THREADS + (int)threadIdx.x < total; }
    // element offset of item j from `base`; `dup`: its first elements that the chunk before holds as well
    __device__ __forceinline__ int64_t at(int j, int &dup) const
    {
        const int i = min(j * THREADS + (int)threadIdx.x, total - 1);
        const int p = g.G ? div_by(i, (int)g.cpp, g.m_cpp) : 0;
        const int64_t first = (g.G ? i - p * (int)g.cpp : c0 + i) * E, start = RAG ? min(first, g.HW - E) : first;
        dup = (int)(first - start);
        return (int64_t)p * g.C * g.HW + start;
    }
};

// grid: (segments, C).
template <typename XT, int NJ, bool RAG>
__global__ __launch_bounds__(256) void bn_partial_kernel(const XT *__restrict__ x, float *__restrict__ partial, BnGeom g)
{
    constexpr int E = Elem<XT>::kPerChunk;
    __shared__ float red[4];
    const int s = blockIdx.x, c = blockIdx.y;
    const BnItems<XT, NJ, RAG> items(g, c, s);
    const XT *xp = x + items.base;
    uint4_t raw[NJ];
    int dup[NJ];
    // straight-line loads from clamped addresses, all in flight together (with a bounds test around each load the compiler
    // waits for the loads two at a time); plain (cacheable) ones: what the last-level cache keeps of x is read
    // from there by the apply kernel (8x64x300x300 fp32: 107 -> 89 us)
#pragma unroll
    for (int j = 0; j < NJ; ++j) raw[j] = load_chunk<RAG>(xp + items.at(j, dup[j]));
    float v[NJ][E];
    auto reduce = [&](auto masked) {
        constexpr bool kMasked = decltype(masked)::value;
        auto counts = [&](int j, int e) { return !kMasked || (items.valid(j) && (!RAG || e >= dup[j])); };
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            Elem<XT>::unpack(raw[j], v[j]);
#pragma unroll
            for (int e = 0; e < E; ++e) sum += counts(j, e) ? v[j][e] : 0.f;
        }
        const float len = (float)g.count(s), inv = 1.0f / len;
        const float mean0 = bn_block_sum(sum, red) * inv;
        float s1 = 0.f, s2 = 0.f;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const float d = counts(j, e) ? v[j][e] - mean0 : 0.f;
                s1 += d;
                s2 = __builtin_fmaf(d, d, s2);
            }
        s1 = bn_block_sum(s1, red);
        s2 = bn_block_sum(s2, red);
        if (threadIdx.x == 0) {
            const float dm = s1 * inv;
            // segment statistics: mean = mean0 + dm (kept as two floats), M2 = sum (x - mean)^2
            float *p = partial + ((int64_t)c * g.segs + s) * 3;
            p[0] = mean0;
            p[1] = dm;
            p[2] = __builtin_fmaxf(__builtin_fmaf(-dm * len, dm, s2), 0.f);
        }
    };
    if (!RAG && items.all()) reduce(std::false_type{});
    else reduce(std::true_type{});
}

// grid: C workgroups.  coef[c] = rstd*gamma, coef[C + c] = mean.
template <typename PT>
__global__ __launch_bounds__(256) void bn_finalize_kernel(const float *__restrict__ partial, const PT *__restrict__ gamma,
                                                          float *__restrict__ coef, float *__restrict__ mean_out,
                                                          float *__restrict__ rstd_out, BnGeom g, float eps)
{
    __shared__ double sh_n[256], sh_mean[256], sh_m2[256];
    const int c = blockIdx.x;
    const float *p = partial + (int64_t)c * g.segs * 3;
    // each thread folds its share of the segments in order, then a tree over the threads
    double cnt = 0.0, mean = 0.0, m2 = 0.0;
    for (int i = threadIdx.x; i < g.segs; i += 256) {
        const double nb = (double)g.count(i);
        const double mb = (double)p[3 * i] + (double)p[3 * i + 1], qb = (double)p[3 * i + 2];
        const double nn = cnt + nb, delta = mb - mean;
        mean += delta * (nb / nn);
        m2 += qb + delta * delta * (cnt * nb / nn);
        cnt = nn;
    }
    sh_n[threadIdx.x] = cnt;
    sh_mean[threadIdx.x] = mean;
    sh_m2[threadIdx.x] = m2;
    __syncthreads();
    for (int step = 128; step > 0; step >>= 1) {
        if (threadIdx.x < step) {
            const double na = sh_n[threadIdx.x], nb = sh_n[threadIdx.x + step];
            if (nb > 0.0) {
                const double nn = na + nb, delta = sh_mean[threadIdx.x + step] - sh_mean[threadIdx.x];
                sh_mean[threadIdx.x] += delta * (nb / nn);
                sh_m2[threadIdx.x] += sh_m2[threadIdx.x + step] + delta * delta * (na * nb / nn);
                sh_n[threadIdx.x] = nn;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double var = sh_m2[0] / sh_n[0];
        const float mu = (float)sh_mean[0];
        const float rstd = (float)(1.0 / sqrt(var + (double)eps));
        coef[c] = rstd * Elem<PT>::load1(gamma + c);
        coef[g.C + c] = mu;
        if (mean_out) mean_out[c] = mu;
        if (rstd_out) rstd_out[c] = rstd;
    }
}

template <int THREADS = 256>
__device__ __forceinline__ double bn_block_sum_f64(double v, double *red)
{
#pragma unroll
    for (int step = 32; step > 0; step >>= 1) v += __shfl_xor(v, step);
    __syncthreads();  // red may still be read from the previous use
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double sum = (red[0] + red[1]) + (red[2] + red[3]);
#pragma unroll
    for (int w = 4; w < THREADS / 64; w += 4) sum += (red[w] + red[w + 1]) + (red[w + 2] + red[w + 3]);
    return sum;
}

// Statistics of channel c from its segments' (mean, M2), at most kBnFuseSegs = one per thread:
// mean = sum n_i m_i / n, M2 = sum (M2_i + n_i (m_i - mean)^2), in double.
__device__ __forceinline__ void bn_channel_stats(const float *partial, int c, const BnGeom &g, float eps, double *red, float &mu,
                                                 float &rstd)
{
    static_assert(kBnFuseSegs == 256, "one segment per thread");
    const int i = threadIdx.x;
    const bool in = i < g.segs;
    const float *p = partial + ((int64_t)c * g.segs + (in ? i : 0)) * 3;
    const double nb = in ? (double)g.count(i) : 0.0, mb = (double)p[0] + (double)p[1], qb = in ? (double)p[2] : 0.0;
    const double n = (double)g.N * (double)g.HW, mean = bn_block_sum_f64(nb * mb, red) / n;
    const double var = bn_block_sum_f64(qb + nb * (mb - mean) * (mb - mean), red) / n;
    mu = (float)mean;
    rstd = (float)(1.0 / sqrt(var + (double)eps));
}

// grid: (segments, C).  STATS: the channel's statistics are made here from the segments' (partial, and gamma,
// mean_out, rstd_out, eps with them): 8x64x300x300 fp32 94 -> 88 us with the launch that made them gone; else coef
// holds them.
template <typename XT, typename PT, typename YT, int NJ, bool RAG, bool STATS>
__global__ __launch_bounds__(256) void bn_apply_kernel(const XT *__restrict__ x, const PT *__restrict__ gamma,
                                                       const PT *__restrict__ beta, const float *__restrict__ partial,
                                                       const float *__restrict__ coef, YT *__restrict__ y,
                                                       float *__restrict__ mean_out, float *__restrict__ rstd_out, BnGeom g,
                                                       float eps)
{
    constexpr int E = Elem<XT>::kPerChunk;
    __shared__ double red[4];
    const int s = blockIdx.x, c = blockIdx.y;
    const BnItems<XT, NJ, RAG> items(g, c, s);
    const XT *xp = x + items.base;
    YT *yp = y + items.base;
    uint4_t raw[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        int dup;
        raw[j] = load_chunk_nt<RAG>(xp + items.at(j, dup));
    }
    float scale, mu;
    const float b = Elem<PT>::load1(beta + c);
    if constexpr (STATS) {  // (while the loads fly)
        float rstd;
        bn_channel_stats(partial, c, g, eps, red, mu, rstd);
        scale = rstd * Elem<PT>::load1(gamma + c);
        if (s == 0 && threadIdx.x == 0) {
            if (mean_out) mean_out[c] = mu;
            if (rstd_out) rstd_out[c] = rstd;
        }
    } else {
        scale = coef[c];
        mu = coef[g.C + c];
    }
    auto write = [&](auto masked) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            int dup;
            const int64_t o = items.at(j, dup);
            float v[E], r[E];
            Elem<XT>::unpack(raw[j], v);
#pragma unroll
            for (int e = 0; e < E; ++e) r[e] = __builtin_fmaf(v[e] - mu, scale, b);
            if constexpr (!decltype(masked)::value) {
                store_row_chunk<RAG, YT, E>(yp + o, r);
            } else if (items.valid(j)) {
                // (y may be x: the elements shared with the chunk before may have been overwritten when this one was read,
                // so only that chunk writes them)
                if (!RAG || dup == 0) {
                    store_row_chunk<RAG, YT, E>(yp + o, r);
                } else {
#pragma unroll
                    for (int e = 1; e < E; ++e)
                        if (e >= dup) Elem<YT>::store1(yp + o + e, r[e]);
                }
            }
        }
    };
    // full segment (uniform): straight-line code; with bounds tests the compiler puts a full
    // wait in front of every store, so each store waits for the one before it
    if (!RAG && items.all()) write(std::false_type{});
    else write(std::true_type{});
}

// Channels of up to 4096 chunks (but see `spread` in launch_bn), which a workgroup holds in registers: a workgroup per channel, one launch, x is read once.
// Bound by latency (launch, loads, block sums, stores) and the vector work of one CU per channel; two launches took (us, now):
// 8x232x128x8 bf16 9.5 (4.3), 32x256x7x7 fp32 8.1 (4.2), 8x224x76x16 fp32 10.2 (6.4), 1x40x104x286 bf16 8.6 (6.5).  Larger channels
// use more CUs in two launches (16x39x65x42 bf16, 5472 chunks, 8.1 against 11.0; 10x16x12x194 fp32, 5820, 6.9 against 7.4).
// Sums as in bn_partial_kernel, the waves' in double.
template <typename XT, typename PT, typename YT, int NJ, bool RAG, int THREADS>
__global__ __launch_bounds__(THREADS) void bn_channel_kernel(const XT *__restrict__ x, const PT *__restrict__ gamma,
                                                             const PT *__restrict__ beta, YT *__restrict__ y,
                                                             float *__restrict__ mean_out, float *__restrict__ rstd_out, BnGeom g,
                                                             float eps)
{
    constexpr int E = Elem<XT>::kPerChunk, W = THREADS / 64;
    __shared__ double red[3][W];
    const int c = blockIdx.x;
    const BnItems<XT, NJ, RAG, THREADS> items(g, c, 0);
    const XT *xp = x + items.base;
    uint4_t raw[NJ];
    int dup[RAG ? NJ : 1];
#pragma unroll
    for (int j = 0; j < NJ; ++j) raw[j] = load_chunk_nt<RAG>(xp + items.at(j, dup[RAG ? j : 0]));
    const float b = Elem<PT>::load1(beta + c), w = Elem<PT>::load1(gamma + c);
    const double n = (double)g.N * (double)g.HW;
    float mu, scale, rstd;
    auto block_sum = [&](float v, double *to) {
        v = wave_allreduce(v, OpSum{});
        if ((threadIdx.x & 63) == 0) to[threadIdx.x >> 6] = (double)v;
    };
    auto total = [&](const double *from) {
        double sum = from[0];
#pragma unroll
        for (int i = 1; i < W; ++i) sum += from[i];
        return sum;
    };
    auto reduce = [&](auto masked) {
        constexpr bool kMasked = decltype(masked)::value;
        auto counts = [&](int j, int e) { return !kMasked || (items.valid(j) && (!RAG || e >= dup[RAG ? j : 0])); };
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            float v[E];
            Elem<XT>::unpack(raw[j], v);
#pragma unroll
            for (int e = 0; e < E; ++e) sum += counts(j, e) ? v[e] : 0.f;
        }
        block_sum(sum, red[0]);
        __syncthreads();
        float mean0;
        double dm, var;
        auto moments = [&]() {
            float s1 = 0.f, s2 = 0.f;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                float v[E], q1 = 0.f, q2 = 0.f;  // (chunk by chunk: short chains of roundings)
                Elem<XT>::unpack(raw[j], v);
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const float d = counts(j, e) ? v[e] - mean0 : 0.f;
                    q1 += d;
                    q2 = __builtin_fmaf(d, d, q2);
                }
                s1 += q1;
                s2 += q2;
            }
            block_sum(s1, red[1]);
            block_sum(s2, red[2]);
            __syncthreads();
            dm = total(red[1]) / n;
            const double m2 = total(red[2]) - dm * dm * n;
            var = m2 > 0.0 ? m2 / n : m2 * 0.0;  // (NaN stays)
        };
        // 16 bits of the mean: the differences of bf16 elements are exact then (one rounding pattern for a whole channel would
        // not average out).  Where they miss it by more than half a deviation (fp32, a mean of 3e4 deviations and more) var
        // would be what cancellation leaves of m2, so again about the mean itself: relative error of var at mean / deviation
        // 1e6 1.5e-5 without, under 1e-7 with.  (dm and var are the same in all threads.)
        mean0 = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, (float)(total(red[0]) / n)) & 0xffffff00u);
        moments();
        if (__builtin_amdgcn_readfirstlane(4.0 * dm * dm > var)) {
            mean0 = (float)((double)mean0 + dm);
            __syncthreads();  // (the sums have been read)
            moments();
        }
        mu = (float)((double)mean0 + dm);
        rstd = (float)(1.0 / sqrt(var + (double)eps));
    };
    if (!RAG && items.all()) reduce(std::false_type{});
    else reduce(std::true_type{});
    scale = rstd * w;
    if (threadIdx.x == 0) {
        if (mean_out) mean_out[c] = mu;
        if (rstd_out) rstd_out[c] = rstd;
    }
    // (y may be x: everything has been read.  Elements that two chunks of a ragged plane share are written twice, the same.)
    YT *yp = y + items.base;
    auto write = [&](auto masked) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            int skip;
            const int64_t o = items.at(j, skip);
            float v[E], r[E];
            Elem<XT>::unpack(raw[j], v);
#pragma unroll
            for (int e = 0; e < E; ++e) r[e] = __builtin_fmaf(v[e] - mu, scale, b);
            if (!decltype(masked)::value || items.valid(j)) store_row_chunk<RAG, YT, E>(yp + o, r);
        }
    };
    if (!RAG && items.all()) write(std::false_type{});
    else write(std::true_type{});
}

// Planes of fewer elements than a chunk of 16 bytes: a workgroup per channel, an element at a time, sums in double.
template <typename XT, typename PT, typename YT, int THREADS>
__global__ __launch_bounds__(THREADS) void bn_small_kernel(const XT *__restrict__ x, const PT *__restrict__ gamma,
                                                       const PT *__restrict__ beta, YT *__restrict__ y,
                                                       float *__restrict__ mean_out, float *__restrict__ rstd_out, int HW, int C,
                                                       int N, float eps)
{
    __shared__ double red[THREADS / 64];
    const int c = blockIdx.x, total = N * HW;
    auto at = [&](int i) { return ((int64_t)(i / HW) * C + c) * HW + i % HW; };
    double sum = 0.0, sq = 0.0;
#pragma unroll(THREADS == 1024 ? 4 : 1)
    for (int i = threadIdx.x; i < total; i += THREADS) sum += (double)Elem<XT>::load1(x + at(i));
    const double mean = bn_block_sum_f64<THREADS>(sum, red) / total;
#pragma unroll(THREADS == 1024 ? 4 : 1)
    for (int i = threadIdx.x; i < total; i += THREADS) {
        const double d = (double)Elem<XT>::load1(x + at(i)) - mean;
        sq += d * d;
    }
    const float mu = (float)mean, rstd = (float)(1.0 / sqrt(bn_block_sum_f64<THREADS>(sq, red) / total + (double)eps));
    const float scale = rstd * Elem<PT>::load1(gamma + c), b = Elem<PT>::load1(beta + c);
    if (threadIdx.x == 0) {
        if (mean_out) mean_out[c] = mu;
        if (rstd_out) rstd_out[c] = rstd;
    }
#pragma unroll(THREADS == 1024 ? 4 : 1)
    for (int i = threadIdx.x; i < total; i += THREADS)
        Elem<YT>::store1(y + at(i), __builtin_fmaf(Elem<XT>::load1(x + at(i)) - mu, scale, b));
}

struct BnArgs {
    const void *x, *gamma, *beta;
    void *y;
    float *mean_out, *rstd_out, *ws;
    int64_t N, C, HW;
    float eps;
    hipStream_t st;
};

// Where a channel is cut: whole segments of 16384 elements from planes of more than half of that; smaller planes in
// groups, as many to a segment as leave about 1024 workgroups (32x256x7x7 fp32 in one workgroup per plane took 38 us).
static BnGeom bn_geom(const BnArgs &a, int E)
{
    BnGeom g{a.HW, (int)a.C, (int)a.N, (a.HW + E - 1) / E, 0, 1, 0, 0};
    if (a.HW > kBnSeg / 2) {
        g.spp = (int)((a.HW + kBnSeg - 1) / kBnSeg);
        g.segs = g.N * g.spp;
    } else {
        int64_t most = (kBnSeg / E) / g.cpp, want = a.N * a.C / 1024;
        if (want > most) want = most;
        if (want > a.N) want = a.N;
        g.G = want < 1 ? 1 : (int)want;
        g.segs = (g.N + g.G - 1) / g.G;
        g.m_cpp = div_magic(g.cpp);
    }
    return g;
}

template <typename XT, typename PT, typename YT, int NJ, bool RAG>
static void launch_bn_nj(const BnArgs &a, const BnGeom &g)
{
    float *partial = a.ws, *coef = a.ws + (int64_t)3 * a.C * g.segs;
    const dim3 grid((unsigned)g.segs, (unsigned)a.C);
    hipLaunchKernelGGL((bn_partial_kernel<XT, NJ, RAG>), grid, dim3(256), 0, a.st, (const XT *)a.x, partial, g);
    const bool fuse = g.segs <= kBnFuseSegs;
    if (!fuse)
        hipLaunchKernelGGL((bn_finalize_kernel<PT>), dim3((unsigned)a.C), dim3(256), 0, a.st, partial, (const PT *)a.gamma, coef,
                           a.mean_out, a.rstd_out, g, a.eps);
    auto kern = fuse ? bn_apply_kernel<XT, PT, YT, NJ, RAG, true> : bn_apply_kernel<XT, PT, YT, NJ, RAG, false>;
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, a.st, (const XT *)a.x, (const PT *)a.gamma, (const PT *)a.beta, partial, coef,
                       (YT *)a.y, a.mean_out, a.rstd_out, g, a.eps);
}

template <typename XT, typename PT, typename YT>
static void launch_bn(const BnArgs &a, bool vec)
{
    constexpr int E = Elem<XT>::kPerChunk;
    if (a.HW < E) {
        // (a few channels with many elements: 1 x (60000 planes of 7) bf16 287 us with 1024 threads, 758 with 256; a workgroup per
        // plane and a merge took 295)
        const bool many = a.N * a.HW > 8192;
        const int threads = many ? 1024 : 256;
        auto kern = many ? bn_small_kernel<XT, PT, YT, 1024> : bn_small_kernel<XT, PT, YT, 256>;
        hipLaunchKernelGGL(kern, dim3((unsigned)a.C), dim3(threads), 0, a.st, (const XT *)a.x,
                           (const PT *)a.gamma, (const PT *)a.beta, (YT *)a.y, a.mean_out, a.rstd_out, (int)a.HW, (int)a.C,
                           (int)a.N, a.eps);
        return;
    }
    const int64_t cpp = (a.HW + E - 1) / E;
    // (bf16 has twice the elements to a chunk, and ragged ones are masked one by one: with few planes, each a small workgroup's, two launches
    // share that among more CUs.  us, one launch, two: 32x16x7x127 8.4, 6.6; 37x4x7x101 7.6, 6.2; 16x8x112x18 6.5, 5.8; but with
    // 2000 ragged chunks 0.86 of the two, 3500 whole ones 0.98, more than 512 planes 0.9, 7x48x32x136 with 544 chunks in each 6.5, 7.6)
    const bool spread = E == 8 && a.N * cpp > (vec ? 3520 : 2048) && a.N * a.C <= 512 && cpp <= (vec ? 256 : 560);
    if (a.N * cpp <= 4096 && !spread) {
        const BnGeom g{a.HW, (int)a.C, (int)a.N, cpp, (int)a.N, 0, 1, div_magic(cpp)};
        auto go = [&](auto nj, auto threads) {
            constexpr int NJ = decltype(nj)::value, THREADS = decltype(threads)::value;
            auto kern = vec ? bn_channel_kernel<XT, PT, YT, NJ, false, THREADS> : bn_channel_kernel<XT, PT, YT, NJ, true, THREADS>;
            hipLaunchKernelGGL(kern, dim3((unsigned)a.C), dim3(THREADS), 0, a.st, (const XT *)a.x, (const PT *)a.gamma, (const PT *)a.beta,
                               (YT *)a.y, a.mean_out, a.rstd_out, g, a.eps);
        };
        const int64_t items = a.N * cpp;
        if (items <= 256) go(std::integral_constant<int, 1>{}, std::integral_constant<int, 256>{});
        else if (items <= 1024) go(std::integral_constant<int, 4>{}, std::integral_constant<int, 256>{});
        else if (items <= 2048) go(std::integral_constant<int, 2>{}, std::integral_constant<int, 1024>{});
        else go(std::integral_constant<int, 4>{}, std::integral_constant<int, 1024>{});
        return;
    }
    const BnGeom g = bn_geom(a, E);
    const int64_t items = g.G ? g.G * g.cpp : g.cpp < kBnSeg / E ? g.cpp : kBnSeg / E, slots = (items + 255) / 256;
    auto go = [&](auto nj) {
        constexpr int NJ = decltype(nj)::value;
        if (vec) launch_bn_nj<XT, PT, YT, NJ, false>(a, g);
        else launch_bn_nj<XT, PT, YT, NJ, true>(a, g);
    };
    if (slots <= 1) go(std::integral_constant<int, 1>{});
    else if (slots <= 2) go(std::integral_constant<int, 2>{});
    else if (slots <= 4) go(std::integral_constant<int, 4>{});
    else if (slots <= 8) go(std::integral_constant<int, 8>{});
    else if constexpr (E == 4) go(std::integral_constant<int, 16>{});
}

template <typename XT, typename PT>
static void launch_bn_y(const BnArgs &a, bool vec, int y_dt)
{
    if (y_dt == PERF_F32) launch_bn<XT, PT, float>(a, vec);
    else launch_bn<XT, PT, uint16_t>(a, vec);
}

static bool bn_shape_ok(int64_t N, int64_t C, int64_t H, int64_t W)
{
    const int64_t kDim = 1 << 24;
    if (N < 1 || C < 1 || H < 1 || W < 1 || N > kDim || C > kDim || H > kDim || W > kDim) return false;
    const int64_t HW = H * W;
    if (N * C > kMaxGridYZ || N * C > (INT64_MAX / 8) / HW) return false;  // planes ride on grid.y
    return true;
}

}  // namespace perf

extern "C" int64_t perf_batchnorm_workspace_bytes(int64_t N, int64_t C, int64_t H, int64_t W)
{
    using namespace perf;
    if (!bn_shape_ok(N, C, H, W)) return -1;
    const int64_t segs = (H * W + kBnSeg - 1) / kBnSeg;
    return 4 * (3 * C * N * segs + 2 * C);
}

namespace perf {

// Scratch of perf_batchnorm_static: the segment partials and the per-channel coefficients that
// perf_batchnorm keeps in the caller's workspace.  One copy per GPU, held until the process ends.
constexpr int64_t kBnStaticFloats = 65536;  // 256 KiB
static __device__ __align__(256) float bn_static_scratch[kBnStaticFloats];

constexpr int kBnMaxDevices = 64;
static std::atomic<float *> bn_static_ptr[kBnMaxDevices];

// Device address of this GPU's copy of the array (the array's name is only a host-side handle).
// Looked up once per device, with that device current; no allocation is involved.
static float *bn_static_address()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kBnMaxDevices) return nullptr;
    float *p = bn_static_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        void *sym = nullptr;
        if (hipGetSymbolAddress(&sym, HIP_SYMBOL(bn_static_scratch)) != hipSuccess || !sym) return nullptr;
        p = static_cast<float *>(sym);
        bn_static_ptr[dev].store(p, std::memory_order_release);  // every thread computes the same value
    }
    return p;
}

}  // namespace perf

namespace perf {

// Host-side argument checks shared by both entry points (no HIP call).
static perf_status bn_check(const void *x, const void *gamma, const void *beta, const void *y, const float *mean_out,
                            const float *rstd_out, int64_t N, int64_t C, int64_t H, int64_t W, float eps, int x_dt,
                            int param_dt, int y_dt)
{
    if (!x || !gamma || !beta || !y) return PERF_ERR_NULL;
    if (!dtype_ok(x_dt) || !dtype_ok(param_dt) || !dtype_ok(y_dt)) return PERF_ERR_DTYPE;
    if (!bn_shape_ok(N, C, H, W) || !(eps >= 0.f) || !std::isfinite(eps)) return PERF_ERR_SHAPE;
    if (!aligned(x, dtype_size(x_dt)) || !aligned(y, dtype_size(y_dt)) || !aligned(gamma, dtype_size(param_dt)) ||
        !aligned(beta, dtype_size(param_dt)) || (mean_out && !aligned(mean_out, 4)) || (rstd_out && !aligned(rstd_out, 4)))
        return PERF_ERR_ALIGN;
    return PERF_OK;
}

static perf_status bn_run(const void *x, const void *gamma, const void *beta, void *y, float *mean_out, float *rstd_out,
                          float *workspace, int64_t N, int64_t C, int64_t H, int64_t W, float eps, int x_dt, int param_dt,
                          int y_dt, perf_stream stream)
{
    const int64_t HW = H * W, ex = 16 / dtype_size(x_dt);
    // 16-byte path: every plane starts 16-byte aligned in x and y, and holds whole chunks
    const bool vec = HW % ex == 0 && aligned(x, 16) && aligned(y, 16) && (HW * dtype_size(y_dt)) % 16 == 0;
    BnArgs a{x, gamma, beta, y, mean_out, rstd_out, workspace, N, C, HW, eps, static_cast<hipStream_t>(stream)};
    if (x_dt == PERF_F32) {
        if (param_dt == PERF_F32) launch_bn_y<float, float>(a, vec, y_dt);
        else launch_bn_y<float, uint16_t>(a, vec, y_dt);
    } else {
        if (param_dt == PERF_F32) launch_bn_y<uint16_t, float>(a, vec, y_dt);
        else launch_bn_y<uint16_t, uint16_t>(a, vec, y_dt);
    }
    return launch_status();
}

}  // namespace perf

extern "C" perf_status perf_batchnorm(const void *x, const void *gamma, const void *beta, void *y, float *mean_out,
                                      float *rstd_out, void *workspace, int64_t N, int64_t C, int64_t H, int64_t W,
                                      float eps, perf_dtype x_dt, perf_dtype param_dt, perf_dtype y_dt, perf_stream stream)
{
    using namespace perf;
    if (!workspace) return PERF_ERR_NULL;
    const perf_status s = bn_check(x, gamma, beta, y, mean_out, rstd_out, N, C, H, W, eps, x_dt, param_dt, y_dt);
    if (s != PERF_OK) return s;
    if (!aligned(workspace, 4)) return PERF_ERR_ALIGN;
    return bn_run(x, gamma, beta, y, mean_out, rstd_out, static_cast<float *>(workspace), N, C, H, W, eps, x_dt, param_dt,
                  y_dt, stream);
}

extern "C" int64_t perf_batchnorm_static_max_bytes(void) { return 4 * perf::kBnStaticFloats; }

extern "C" perf_status perf_batchnorm_static(const void *x, const void *gamma, const void *beta, void *y,
                                             float *mean_out, float *rstd_out, int64_t N, int64_t C, int64_t H,
                                             int64_t W, float eps, perf_dtype x_dt, perf_dtype param_dt,
                                             perf_dtype y_dt, perf_stream stream)
{
    using namespace perf;
    const perf_status s = bn_check(x, gamma, beta, y, mean_out, rstd_out, N, C, H, W, eps, x_dt, param_dt, y_dt);
    if (s != PERF_OK) return s;
    if (perf_batchnorm_workspace_bytes(N, C, H, W) > perf_batchnorm_static_max_bytes())
        return PERF_ERR_UNSUPPORTED;  // the problem needs more scratch than the built-in array holds
    float *scratch = bn_static_address();  // first HIP call: every check above ran without one
    if (!scratch) return PERF_ERR_LAUNCH;
    return bn_run(x, gamma, beta, y, mean_out, rstd_out, scratch, N, C, H, W, eps, x_dt, param_dt, y_dt, stream);
}
