// Streaming operators of the paper's operator table (Section 4.3) beyond softmax and
// LayerNorm: RMS normalisation ("rmsnorm"), the mean along an axis ("reducemean") and the
// element-wise "add" / "mul" / "relu".  All are bound by HBM; each reads its input once with
// 16-byte accesses and writes once.  No atomics, no workspace.
//
//  * rmsnorm_rows_kernel: a wavefront owns a row (as in LayerNorm): one load of the row into
//    registers, sum of squares by a DPP / permlane butterfly, scale, 16-byte stores; gamma is
//    staged once per workgroup in LDS.  rmsnorm_block_kernel: general fallback.
//  * rowmean_kernel: a wavefront per row, any length.
//  * colmean_kernel: a workgroup owns 4 or 8 chunks of 16 bytes of every row (64 or 128
//    contiguous bytes per row); 64 or 32 row lanes stride over the rows and are combined
//    through LDS; workgroups that share 128-byte lines are placed on the same XCD.
//  * eltwise_kernel: one pass, four 16-byte vectors per thread.
#include "row_io.h"
#include "wide_rows.h"
#include "host_utils.h"
#include <type_traits>

namespace perf {

// ---- RMS norm ------------------------------------------------------------------------
constexpr int kRmsThreads = 256;
constexpr int kRmsWaves = kRmsThreads / 64;

// NC: 16-byte chunks of the row held per lane (cols <= NC * 64 * E); RAG: rows that are no whole aligned chunks (row_io.h).
template <typename XT, typename PT, typename YT, int NC, bool RAG = false>
__global__ __launch_bounds__(kRmsThreads) void rmsnorm_rows_kernel(const XT *__restrict__ x, const PT *__restrict__ gamma,
                                                                   YT *__restrict__ y, float *__restrict__ rrms_out,
                                                                   int64_t rows, int cols, int64_t ldx, int64_t ldy,
                                                                   float eps)
{
    constexpr int E = Elem<XT>::kPerChunk;
    constexpr int NCH = NC * 64;
    // gamma as fp32 in planes of 4 floats per chunk: plane q of chunk c holds elements c*E + 4q .. +3
    extern __shared__ float4_t lds[];
    for (int i = threadIdx.x; i < (E / 4) * NCH; i += kRmsThreads) {
        const int q = i / NCH, c = i % NCH;
        const int col = chunk_start<RAG, E>(c * E, cols) + 4 * q;
        float4_t g = {0.f, 0.f, 0.f, 0.f};
        if (c * E < cols) {
#pragma unroll
            for (int e = 0; e < 4; ++e) g[e] = Elem<PT>::load1(gamma + col + e);
        }
        lds[i] = g;
    }
    __syncthreads();

    const int lane = threadIdx.x & 63;
    const int64_t wave = (int64_t)blockIdx.x * kRmsWaves + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * kRmsWaves;
    const float inv_cols = 1.0f / (float)cols;

    uint4_t raw[NC];
    auto load_row = [&](int64_t r) {
        const XT *xr = x + r * ldx;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int c = (j * 64 + lane) * E;
            raw[j] = c < cols ? load_chunk_nt<RAG>(xr + chunk_start<RAG, E>(c, cols)) : uint4_t{0u, 0u, 0u, 0u};
        }
    };
    if (wave < rows) load_row(wave);
    for (int64_t r = wave; r < rows; r += nwaves) {
        float v[NC][E];
        float ss = 0.f;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            Elem<XT>::unpack(raw[j], v[j]);
#pragma unroll
            for (int e = 0; e < E; ++e) {  // (padding chunks hold zeros)
                const float once = !RAG || e >= (j * 64 + lane) * E - chunk_start<RAG, E>((j * 64 + lane) * E, cols) ? v[j][e] : 0.f;
                ss = __builtin_fmaf(once, once, ss);
            }
        }
        if (r + nwaves < rows) load_row(r + nwaves);  // next row's loads fly during this row's arithmetic
        ss = wave_allreduce(ss, OpSum{});
        const float rr = 1.0f / __builtin_sqrtf(ss * inv_cols + eps);
        if (lane == 0 && rrms_out) rrms_out[r] = rr;
        YT *yr = y + r * ldy;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int ch = j * 64 + lane;
            if (ch * E < cols) {
                float o[E];
#pragma unroll
                for (int q = 0; q < E / 4; ++q) {
                    const float4_t g = lds[q * NCH + ch];
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[4 * q + e] = v[j][4 * q + e] * rr * g[e];
                }
                store_row_chunk<RAG, YT, E>(yr + chunk_start<RAG, E>(ch * E, cols), o);
            }
            __builtin_amdgcn_sched_barrier(0);  // keeps the gamma reads chunk by chunk (register count)
        }
    }
}

__device__ __forceinline__ float block_sum_256(float v, float *red)
{
    v = wave_allreduce(v, OpSum{});
    __syncthreads();  // red may still be read from the previous use
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// General fallback: one workgroup per row, scalar accesses, two passes.
template <typename XT, typename PT, typename YT>
__global__ __launch_bounds__(256) void rmsnorm_block_kernel(const XT *__restrict__ x, const PT *__restrict__ gamma,
                                                            YT *__restrict__ y, float *__restrict__ rrms_out,
                                                            int64_t rows, int64_t cols, int64_t ldx, int64_t ldy,
                                                            float eps)
{
    __shared__ float red[4];
    for (int64_t r = blockIdx.x; r < rows; r += gridDim.x) {
        const XT *xr = x + r * ldx;
        float ss = 0.f;
        for (int64_t c = threadIdx.x; c < cols; c += 256) {
            const float v = Elem<XT>::load1(xr + c);
            ss = __builtin_fmaf(v, v, ss);
        }
        const float rr = 1.0f / __builtin_sqrtf(block_sum_256(ss, red) / (float)cols + eps);
        if (threadIdx.x == 0 && rrms_out) rrms_out[r] = rr;
        for (int64_t c = threadIdx.x; c < cols; c += 256)
            Elem<YT>::store1(y + r * ldy + c, Elem<XT>::load1(xr + c) * rr * Elem<PT>::load1(gamma + c));
    }
}

struct RmsArgs {
    const void *x, *gamma;
    void *y;
    float *rrms;
    int64_t rows, cols, ldx, ldy;
    float eps;
    hipStream_t st;
    bool params_vec;  // gamma is 16-byte aligned
    bool failed;
};

template <typename XT, typename PT, typename YT, int NC, bool RAG = false>
static void launch_rms_nc(const RmsArgs &a)
{
    constexpr int E = Elem<XT>::kPerChunk;
    const size_t lds_bytes = (size_t)(E / 4) * NC * 64 * sizeof(float4_t);
    int64_t blocks = (a.rows + kRmsWaves - 1) / kRmsWaves;
    if (blocks > 512) blocks = 512;  // two workgroups per CU; waves then loop over rows
    hipLaunchKernelGGL((rmsnorm_rows_kernel<XT, PT, YT, NC, RAG>), dim3((unsigned)blocks), dim3(kRmsThreads), lds_bytes, a.st,
                       (const XT *)a.x, (const PT *)a.gamma, (YT *)a.y, a.rrms, a.rows, (int)a.cols, a.ldx, a.ldy, a.eps);
}

template <typename XT, typename PT, typename YT>
static void launch_rms_typed(RmsArgs &a, bool vec_ok)
{
    constexpr int E = Elem<XT>::kPerChunk;
    const int64_t chunks = (a.cols + 64 * E - 1) / (64 * E);
    if (vec_ok && chunks <= 16) {
        if (chunks <= 2) launch_rms_nc<XT, PT, YT, 2>(a);
        else if (chunks <= 8) launch_rms_nc<XT, PT, YT, 8>(a);
        else launch_rms_nc<XT, PT, YT, 16>(a);
    } else if (vec_ok && a.params_vec) {
        // longer rows: a workgroup per row, the row parked in LDS (one read of HBM)
        a.failed = launch_norm_wide<XT, PT, YT, true>(a.x, a.gamma, a.gamma, a.y, nullptr, a.rrms, a.rows, a.cols, a.ldx,
                                                      a.ldy, a.eps, a.st) != 0;
    } else if (a.cols >= E && chunks <= (E == 8 ? 16 : 8)) {
        // no whole aligned chunks: the same kernel with ragged ones (20000 x 1999 fp32: 58 us, element accesses in two
        // passes took 108; 9000 x 4999 bf16: 36 us, 42 with a workgroup per row)
        if (chunks <= 2) launch_rms_nc<XT, PT, YT, 2, true>(a);
        else if (chunks <= 4) launch_rms_nc<XT, PT, YT, 4, true>(a);
        else if (chunks <= 8) launch_rms_nc<XT, PT, YT, 8, true>(a);
        else if constexpr (E == 8) launch_rms_nc<XT, PT, YT, 16, true>(a);
    } else if (a.cols >= E && a.cols <= wide_ragged_max<XT>()) {
        launch_norm_ragged<XT, PT, YT, true>(a.x, a.gamma, a.gamma, a.y, nullptr, a.rrms, a.rows, a.cols, a.ldx, a.ldy, a.eps,
                                             a.st);
    } else {
        const int64_t blocks = a.rows < 65536 ? a.rows : 65536;
        hipLaunchKernelGGL((rmsnorm_block_kernel<XT, PT, YT>), dim3((unsigned)blocks), dim3(256), 0, a.st,
                           (const XT *)a.x, (const PT *)a.gamma, (YT *)a.y, a.rrms, a.rows, a.cols, a.ldx, a.ldy, a.eps);
    }
}

template <typename XT, typename PT>
static void launch_rms_y(RmsArgs &a, bool vec_ok, int y_dt)
{
    if (y_dt == PERF_F32) launch_rms_typed<XT, PT, float>(a, vec_ok);
    else launch_rms_typed<XT, PT, uint16_t>(a, vec_ok);
}

template <typename XT>
static void launch_rms_p(RmsArgs &a, bool vec_ok, int p_dt, int y_dt)
{
    if (p_dt == PERF_F32) launch_rms_y<XT, float>(a, vec_ok, y_dt);
    else launch_rms_y<XT, uint16_t>(a, vec_ok, y_dt);
}

// ---- means ---------------------------------------------------------------------------
// Mean of every row: a wavefront per row; 16-byte loads, at the elements' own alignment unless ALIGNED, and the few
// elements that fill no chunk one by one.
// ELEMENTS: short unaligned rows, element loads only (40000 x 129 bf16: 6.6 us, 10.8 with chunks that leave most lanes idle).
template <typename XT, typename YT, bool ALIGNED, bool ELEMENTS = false>
__global__ __launch_bounds__(256) void rowmean_kernel(const XT *__restrict__ x, YT *__restrict__ y, int64_t rows,
                                                      int64_t cols, int64_t ldx)
{
    constexpr int E = Elem<XT>::kPerChunk;
    const int lane = threadIdx.x & 63;
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t r = wave; r < rows; r += nwaves) {
        const XT *xr = x + r * ldx;
        float s0 = 0.f, s1 = 0.f;
        if constexpr (ELEMENTS) {
            for (int64_t c = lane; c < cols; c += 64) s0 += Elem<XT>::load1(xr + c);
        } else {
            const int64_t nch = cols / E;
            int64_t c = lane;
            constexpr int kU = 8;  // eight independent 16-byte loads in flight per lane (8 KiB per wave)
            for (; c + 64 * (kU - 1) < nch; c += 64 * kU) {
                uint4_t raw[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) raw[u] = load_chunk_nt<!ALIGNED>(xr + (c + 64 * u) * E);
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    float v[E];
                    Elem<XT>::unpack(raw[u], v);
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        if (u & 1) s1 += v[e];
                        else s0 += v[e];
                    }
                }
            }
            for (; c + 64 < nch; c += 128) {  // two at a time
                const uint4_t r0 = load_chunk_nt<!ALIGNED>(xr + c * E);
                const uint4_t r1 = load_chunk_nt<!ALIGNED>(xr + (c + 64) * E);
                float v0[E], v1[E];
                Elem<XT>::unpack(r0, v0);
                Elem<XT>::unpack(r1, v1);
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    s0 += v0[e];
                    s1 += v1[e];
                }
            }
            if (c < nch) {
                float v0[E];
                Elem<XT>::unpack(load_chunk_nt<!ALIGNED>(xr + c * E), v0);
#pragma unroll
                for (int e = 0; e < E; ++e) s0 += v0[e];
            }
            if (!ALIGNED && nch * E + lane < cols) s1 += Elem<XT>::load1(xr + nch * E + lane);
        }
        const float s = wave_allreduce(s0 + s1, OpSum{});
        if (lane == 0) Elem<YT>::store1(y + r, s / (float)cols);
    }
}

// Mean of every column, 16-byte path: thread = (row lane tid/CW, chunk tid%CW); a workgroup
// owns CW chunks of 16 bytes (CW * E columns) of every row.  With CW = 8 and 16-byte elements
// groups of 4 the workgroup reads whole 128-byte lines; with CW = 4 two neighbouring
// workgroups share each line, and the group index is remapped so that they run on the same
// XCD (workgroup ids are dealt round-robin to the 8 XCDs, whose L2s are private: without the
// remap both XCDs fetch the line from memory).
// RAG: columns that are no whole aligned chunks (row_io.h), at least one chunk of them.
template <typename XT, typename YT, int CW, int THREADS, bool RAG = false>
__global__ __launch_bounds__(THREADS) void colmean_kernel(const XT *__restrict__ x, YT *__restrict__ y, int64_t rows,
                                                          int64_t cols, int64_t ldx)
{
    constexpr int E = Elem<XT>::kPerChunk;
    constexpr int kRowLanes = THREADS / CW;
    constexpr int kUnroll = 4096 / THREADS;  // 64 KiB in flight per workgroup: 16 x 16 bytes per thread of 256, 4 of 1024
    __shared__ float part[kRowLanes][CW * E + 1];
    const int64_t group = gridDim.x % 8 == 0 ? (int64_t)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3)
                                             : (int64_t)blockIdx.x;
    const int cl = threadIdx.x % CW, rl = threadIdx.x / CW;
    const int64_t col0 = (group * CW + cl) * E;
    float acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0.f;
    if (col0 < cols) {  // (a chunk is entirely valid or not)
        const XT *xc = x + (RAG ? min(col0, cols - E) : col0);
        int64_t r = rl;
        for (; r + kRowLanes * (kUnroll - 1) < rows; r += kRowLanes * kUnroll) {
            uint4_t raw[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) raw[u] = load_chunk_nt<RAG>(xc + (r + kRowLanes * u) * ldx);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                float v[E];
                Elem<XT>::unpack(raw[u], v);
#pragma unroll
                for (int e = 0; e < E; ++e) acc[e] += v[e];
            }
        }
        for (; r < rows; r += kRowLanes) {
            float v[E];
            Elem<XT>::unpack(load_chunk_nt<RAG>(xc + r * ldx), v);
#pragma unroll
            for (int e = 0; e < E; ++e) acc[e] += v[e];
        }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) part[rl][cl * E + e] = acc[e];
    // The row lanes' partial sums of a column are added in rounds of at most 8 terms per thread
    // (one thread adding all kRowLanes of them in a row is 64 .. 256 dependent LDS reads: several
    // microseconds at the end of a 20 us kernel); the order is fixed, so reruns are bit-identical.
    constexpr int kCols = CW * E;
    const int col = threadIdx.x % kCols, grp = threadIdx.x / kCols;
    int n = kRowLanes;  // partial sums per column still to add
    while (n > 1) {
        const int step = n > 8 ? 8 : n, out = (n + step - 1) / step;
        __syncthreads();
        float s = 0.f;
        const bool mine = grp < out;
        if (mine)
            for (int i = grp * step; i < min(n, (grp + 1) * step); ++i) s += part[i][col];
        __syncthreads();
        if (mine) part[grp][col] = s;
        n = out;
    }
    __syncthreads();
    if (threadIdx.x < kCols) {
        // (element e of a chunk that would overhang the columns is column cols - E + e; those that the chunk before has as well
        // are written by that one)
        const int64_t first = group * kCols + threadIdx.x / E * E, start = RAG ? min(first, cols - E) : first;
        const int64_t c = start + threadIdx.x % E;
        if (first < cols && c >= first) Elem<YT>::store1(y + c, part[0][threadIdx.x] / (float)rows);
    }
}

// Mean of every column, element path: a thread per column.
template <typename XT, typename YT>
__global__ __launch_bounds__(256) void colmean_scalar_kernel(const XT *__restrict__ x, YT *__restrict__ y, int64_t rows,
                                                             int64_t cols, int64_t ldx)
{
    const int64_t col = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (col >= cols) return;
    float s = 0.f;
    for (int64_t r = 0; r < rows; ++r) s += Elem<XT>::load1(x + r * ldx + col);
    Elem<YT>::store1(y + col, s / (float)rows);
}

template <typename XT, typename YT>
static void launch_mean(const void *x, void *y, int64_t rows, int64_t cols, int64_t ldx, int axis, hipStream_t st)
{
    constexpr int E = Elem<XT>::kPerChunk;
    const bool vec = cols % E == 0 && ldx % E == 0 && aligned(x, 16);
    if (axis == 1) {
        int64_t blocks = (rows + 3) / 4;
        if (blocks > 256 * 64) blocks = 256 * 64;
        auto kern = vec ? rowmean_kernel<XT, YT, true>
                    : cols < 128 * E ? rowmean_kernel<XT, YT, false, true> : rowmean_kernel<XT, YT, false>;
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, st, (const XT *)x, (YT *)y, rows, cols, ldx);
    } else if (vec) {
        // whole 128-byte lines per workgroup when that still gives every CU a workgroup
        // (fewer, 16-wave workgroups on whole lines, or 32-byte segments for more workgroups, measured
        // no better on 4096 x 4096: 19.5 and 25.7 us against 18.5)
        constexpr int kWide = 8;
        const int64_t nwide = (cols + kWide * E - 1) / (kWide * E);
        if (nwide >= 256)
            hipLaunchKernelGGL((colmean_kernel<XT, YT, kWide, 256>), dim3((unsigned)nwide), dim3(256), 0, st, (const XT *)x,
                               (YT *)y, rows, cols, ldx);
        else
            hipLaunchKernelGGL((colmean_kernel<XT, YT, 4, 256>), dim3((unsigned)((cols + 4 * E - 1) / (4 * E))), dim3(256),
                               0, st, (const XT *)x, (YT *)y, rows, cols, ldx);
    } else if (cols >= E && rows >= 16) {
        // (a few rows stay with a thread per column: 3 x 1001 2.8 us against 3.1, 15 x 100001 3.9 against 6.5;
        // a thread per column, all rows in turn, took 12.4 ms on 51480 x 777 fp32: 168 us; narrower groups where there are few:
        // 9000 x 2222 bf16 36 us against 40, but 5000 x 4001 fp32 55 against 37)
        auto go = [&](auto cw) {
            constexpr int CW = decltype(cw)::value;
            hipLaunchKernelGGL((colmean_kernel<XT, YT, CW, 256, true>), dim3((unsigned)((cols + CW * E - 1) / (CW * E))), dim3(256), 0,
                               st, (const XT *)x, (YT *)y, rows, cols, ldx);
        };
        if (cols >= 128 * 4 * E) go(std::integral_constant<int, 4>{});
        else go(std::integral_constant<int, 2>{});
    } else {
        hipLaunchKernelGGL((colmean_scalar_kernel<XT, YT>), dim3((unsigned)((cols + 255) / 256)), dim3(256), 0, st,
                           (const XT *)x, (YT *)y, rows, cols, ldx);
    }
}

// ---- column mean in two stages (caller-supplied workspace) ----------------------------
// Stage 1: workgroup (cb, sp) sums rows [sp * rows_per, (sp+1) * rows_per) of the 64 chunks
// of 16 bytes starting at chunk cb * 64: a wave reads 1 KiB of one row per instruction, so
// the memory sees long contiguous runs instead of one cache line per row, and the grid is
// as large as the row split makes it, whatever the number of columns.  Stage 2 adds the
// partial sums of a column in split order.  Both orders are fixed: results are reproducible.
constexpr int kColsumTargetGroups = 2048;  // workgroups aimed for in stage 1
constexpr int kColsumMinRows = 32;         // rows per workgroup at least (8 per wave)
constexpr int kColsumUnroll = 8;

struct ColsumPlan {
    int64_t col_blocks, splits, rows_per;
};
static ColsumPlan colsum_plan(int64_t rows, int64_t cols, int E)
{
    ColsumPlan p;
    p.col_blocks = (cols + 64 * E - 1) / (64 * E);
    int64_t splits = (kColsumTargetGroups + p.col_blocks - 1) / p.col_blocks;
    const int64_t max_splits = (rows + kColsumMinRows - 1) / kColsumMinRows;
    if (splits > max_splits) splits = max_splits;
    if (splits < 1) splits = 1;
    p.rows_per = ((rows + splits - 1) / splits + 3) / 4 * 4;
    p.splits = (rows + p.rows_per - 1) / p.rows_per;
    return p;
}

template <typename XT>
__global__ __launch_bounds__(256) void colsum_partial_kernel(const XT *__restrict__ x, float *__restrict__ ws,
                                                             int64_t rows, int64_t cols, int64_t ldx, int64_t rows_per)
{
    constexpr int E = Elem<XT>::kPerChunk;
    __shared__ float part[4][64 * E];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t col0 = ((int64_t)blockIdx.x * 64 + lane) * E;
    const int64_t r0 = (int64_t)blockIdx.y * rows_per;
    const int64_t r1 = r0 + rows_per < rows ? r0 + rows_per : rows;
    float acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0.f;
    if (col0 < cols) {  // cols is a multiple of E
        const XT *xc = x + col0;
        int64_t r = r0 + wave;
        for (; r + 4 * (kColsumUnroll - 1) < r1; r += 4 * kColsumUnroll) {
            uint4_t raw[kColsumUnroll];
#pragma unroll
            for (int u = 0; u < kColsumUnroll; ++u)
                raw[u] = __builtin_nontemporal_load(reinterpret_cast<const uint4_t *>(xc + (r + 4 * u) * ldx));
#pragma unroll
            for (int u = 0; u < kColsumUnroll; ++u) {
                float v[E];
                Elem<XT>::unpack(raw[u], v);
#pragma unroll
                for (int e = 0; e < E; ++e) acc[e] += v[e];
            }
        }
        for (; r < r1; r += 4) {
            float v[E];
            Elem<XT>::unpack(__builtin_nontemporal_load(reinterpret_cast<const uint4_t *>(xc + r * ldx)), v);
#pragma unroll
            for (int e = 0; e < E; ++e) acc[e] += v[e];
        }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) part[wave][e * 64 + lane] = acc[e];
    __syncthreads();
    for (int i = threadIdx.x; i < 64 * E; i += 256) {
        const int e = i / 64, l = i % 64;
        const int64_t col = ((int64_t)blockIdx.x * 64 + l) * E + e;
        if (col < cols) ws[(int64_t)blockIdx.y * cols + col] = (part[0][i] + part[1][i]) + (part[2][i] + part[3][i]);
    }
}

// Stage 2 (1024 threads): thread = (column tid%32 of the block, split lane tid/32): a row of 32 lanes reads
// one 128-byte line of a split's partial sums; a lane has 8 independent loads in flight
// (splits sl, sl+32, .. in batches of 8); the 32 split lanes are combined through LDS in
// lane order.
template <typename YT>
__global__ __launch_bounds__(1024) void colsum_final_kernel(const float *__restrict__ ws, YT *__restrict__ y,
                                                           int64_t rows, int64_t cols, int64_t splits)
{
    constexpr int kLanes = 32, kBatch = 8;
    __shared__ float part[kLanes][32 + 1];
    const int cl = threadIdx.x & 31, sl = threadIdx.x >> 5;
    const int64_t col = (int64_t)blockIdx.x * 32 + cl;
    float s = 0.f;
    if (col < cols) {
        for (int64_t sp = sl; sp < splits; sp += kLanes * kBatch) {
            float v[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) v[u] = sp + u * kLanes < splits ? ws[(sp + u * kLanes) * cols + col] : 0.f;
#pragma unroll
            for (int u = 0; u < kBatch; ++u) s += v[u];
        }
    }
    part[sl][cl] = s;
    __syncthreads();
    if (sl == 0 && col < cols) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < kLanes; ++i) t += part[i][cl];
        Elem<YT>::store1(y + col, t / (float)rows);
    }
}

template <typename XT, typename YT>
static void launch_colmean_ws(const void *x, void *y, float *ws, int64_t rows, int64_t cols, int64_t ldx, hipStream_t st)
{
    constexpr int E = Elem<XT>::kPerChunk;
    const ColsumPlan p = colsum_plan(rows, cols, E);
    hipLaunchKernelGGL((colsum_partial_kernel<XT>), dim3((unsigned)p.col_blocks, (unsigned)p.splits), dim3(256), 0, st,
                       (const XT *)x, ws, rows, cols, ldx, p.rows_per);
    hipLaunchKernelGGL((colsum_final_kernel<YT>), dim3((unsigned)((cols + 31) / 32)), dim3(1024), 0, st, (const float *)ws,
                       (YT *)y, rows, cols, p.splits);
}

// ---- element-wise --------------------------------------------------------------------
template <int OP> __device__ __forceinline__ float apply_op(float a, float b)
{
    if (OP == PERF_ADD) return a + b;
    if (OP == PERF_MUL) return a * b;
    return __builtin_fmaxf(a, 0.f) + 0.f;  // relu; "+ 0" turns a -0 into +0
}

constexpr int kEltUnroll = 4;

// n elements in nvec whole vectors, and the rest one by one by the last workgroup; ALIGNED: 16-byte aligned operands.
template <int OP, typename T, bool ALIGNED>
__global__ __launch_bounds__(256) void eltwise_kernel(const T *__restrict__ a, const T *__restrict__ b, T *__restrict__ y,
                                                      int64_t nvec, int64_t n)
{
    constexpr int E = Elem<T>::kPerChunk;
    const int64_t block0 = (int64_t)blockIdx.x * 256 * kEltUnroll;
    const int64_t base = block0 + threadIdx.x;
    auto av = [&](int64_t i) { return load_chunk_nt<!ALIGNED>(a + i * E); };
    auto bv = [&](int64_t i) { return OP != PERF_RELU ? load_chunk_nt<!ALIGNED>(b + i * E) : uint4_t{0u, 0u, 0u, 0u}; };
    auto combine = [&](const uint4_t &xa, const uint4_t &xb, int64_t i) {
        float va[E], vb[E], o[E];
        Elem<T>::unpack(xa, va);
        if (OP != PERF_RELU) Elem<T>::unpack(xb, vb);
#pragma unroll
        for (int e = 0; e < E; ++e) o[e] = apply_op<OP>(va[e], OP != PERF_RELU ? vb[e] : 0.f);
        store_row_chunk<!ALIGNED, T, E>(y + i * E, o);
    };
    if (blockIdx.x == gridDim.x - 1 && nvec * E + threadIdx.x < n) {  // (fewer than E elements)
        const int64_t i = nvec * E + threadIdx.x;
        Elem<T>::store1(y + i, apply_op<OP>(Elem<T>::load1(a + i), OP != PERF_RELU ? Elem<T>::load1(b + i) : 0.f));
    }
    if (block0 + 256 * kEltUnroll <= nvec) {
        // whole block in range (uniform): straight-line loads, all in flight together.  (With a
        // bounds test around each load the compiler waits for one load before it issues the next.)
        uint4_t ra[kEltUnroll], rb[kEltUnroll];
#pragma unroll
        for (int u = 0; u < kEltUnroll; ++u) {
            ra[u] = av(base + u * 256);
            rb[u] = bv(base + u * 256);
        }
#pragma unroll
        for (int u = 0; u < kEltUnroll; ++u) combine(ra[u], rb[u], base + u * 256);
    } else {
        for (int u = 0; u < kEltUnroll; ++u) {
            const int64_t i = base + u * 256;
            if (i < nvec) combine(av(i), bv(i), i);
        }
    }
}

template <int OP, typename T>
__global__ __launch_bounds__(64) void eltwise_tail_kernel(const T *__restrict__ a, const T *__restrict__ b, T *__restrict__ y,
                                                          int64_t n)
{
    for (int64_t i = threadIdx.x; i < n; i += 64)
        Elem<T>::store1(y + i, apply_op<OP>(Elem<T>::load1(a + i), OP != PERF_RELU ? Elem<T>::load1(b + i) : 0.f));
}

template <int OP, typename T>
static perf_status launch_eltwise(const void *a, const void *b, void *y, int64_t n, hipStream_t st)
{
    constexpr int E = Elem<T>::kPerChunk;
    const bool vec = aligned(a, 16) && aligned(y, 16) && (OP == PERF_RELU || aligned(b, 16));
    if (!vec && n > (int64_t(1) << 20) * 64) return PERF_ERR_UNSUPPORTED;  // (documented limit of misaligned calls)
    const int64_t nvec = n / E;
    if (nvec == 0) {
        hipLaunchKernelGGL((eltwise_tail_kernel<OP, T>), dim3(1), dim3(64), 0, st, (const T *)a,
                           OP != PERF_RELU ? (const T *)b : (const T *)a, (T *)y, n);
        return launch_status();
    }
    const int64_t blocks = (nvec + 256 * kEltUnroll - 1) / (256 * kEltUnroll);
    if (blocks > kMaxGridX) return PERF_ERR_UNSUPPORTED;
    auto kern = vec ? eltwise_kernel<OP, T, true> : eltwise_kernel<OP, T, false>;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, st, (const T *)a, (const T *)b, (T *)y, nvec, n);
    return launch_status();
}

template <typename T>
static perf_status dispatch_eltwise(int op, const void *a, const void *b, void *y, int64_t n, hipStream_t st)
{
    if (op == PERF_ADD) return launch_eltwise<PERF_ADD, T>(a, b, y, n, st);
    if (op == PERF_MUL) return launch_eltwise<PERF_MUL, T>(a, b, y, n, st);
    return launch_eltwise<PERF_RELU, T>(a, b, y, n, st);
}

}  // namespace perf

extern "C" perf_status perf_rmsnorm(const void *x, const void *gamma, void *y, float *rrms_out, int64_t rows,
                                    int64_t cols, int64_t ldx, int64_t ldy, float eps, perf_dtype x_dt,
                                    perf_dtype param_dt, perf_dtype y_dt, perf_stream stream)
{
    using namespace perf;
    if (!x || !gamma || !y) return PERF_ERR_NULL;
    if (!dtype_ok(x_dt) || !dtype_ok(param_dt) || !dtype_ok(y_dt)) return PERF_ERR_DTYPE;
    if (rows < 1 || cols < 1 || ldx < cols || ldy < cols || !(eps >= 0.f) || !std::isfinite(eps)) return PERF_ERR_SHAPE;
    if (rows > (INT64_MAX / 4) / ldx || rows > (INT64_MAX / 4) / ldy) return PERF_ERR_SHAPE;
    if (!aligned(x, dtype_size(x_dt)) || !aligned(y, dtype_size(y_dt)) || !aligned(gamma, dtype_size(param_dt)) ||
        (rrms_out && !aligned(rrms_out, 4)))
        return PERF_ERR_ALIGN;
    const int64_t ex = 16 / dtype_size(x_dt);
    const bool vec_ok = cols % ex == 0 && ldx % ex == 0 && aligned(x, 16) && aligned(y, 16) &&
                        (ldy * dtype_size(y_dt)) % 16 == 0;
    RmsArgs a{x, gamma, y, rrms_out, rows, cols, ldx, ldy, eps, static_cast<hipStream_t>(stream), aligned(gamma, 16), false};
    if (x_dt == PERF_F32) launch_rms_p<float>(a, vec_ok, param_dt, y_dt);
    else launch_rms_p<uint16_t>(a, vec_ok, param_dt, y_dt);
    return a.failed ? PERF_ERR_LAUNCH : launch_status();
}

extern "C" perf_status perf_reduce_mean(const void *x, void *y, int64_t rows, int64_t cols, int64_t ldx, int axis,
                                        perf_dtype x_dt, perf_dtype y_dt, perf_stream stream)
{
    using namespace perf;
    if (!x || !y) return PERF_ERR_NULL;
    if (!dtype_ok(x_dt) || !dtype_ok(y_dt)) return PERF_ERR_DTYPE;
    if (rows < 1 || cols < 1 || ldx < cols || (axis != 0 && axis != 1)) return PERF_ERR_SHAPE;
    if (rows > (INT64_MAX / 4) / ldx || cols > (int64_t)kMaxGridX * 16) return PERF_ERR_SHAPE;
    if (!aligned(x, dtype_size(x_dt)) || !aligned(y, dtype_size(y_dt))) return PERF_ERR_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (x_dt == PERF_F32) {
        if (y_dt == PERF_F32) launch_mean<float, float>(x, y, rows, cols, ldx, axis, st);
        else launch_mean<float, uint16_t>(x, y, rows, cols, ldx, axis, st);
    } else {
        if (y_dt == PERF_F32) launch_mean<uint16_t, float>(x, y, rows, cols, ldx, axis, st);
        else launch_mean<uint16_t, uint16_t>(x, y, rows, cols, ldx, axis, st);
    }
    return launch_status();
}

extern "C" int64_t perf_reduce_mean_workspace_bytes(int64_t rows, int64_t cols, int axis, perf_dtype x_dt)
{
    using namespace perf;
    if (!dtype_ok(x_dt) || rows < 1 || cols < 1 || (axis != 0 && axis != 1)) return -1;
    if (cols > (int64_t)kMaxGridX * 16) return -1;
    const int E = x_dt == PERF_F32 ? 4 : 8;
    if (axis == 1 || cols % E != 0) return 0;
    const ColsumPlan p = colsum_plan(rows, cols, E);
    if (p.splits > 65535) return -1;
    return p.splits * cols * (int64_t)sizeof(float);
}

extern "C" perf_status perf_reduce_mean_ws(const void *x, void *y, void *workspace, int64_t rows, int64_t cols,
                                           int64_t ldx, int axis, perf_dtype x_dt, perf_dtype y_dt, perf_stream stream)
{
    using namespace perf;
    if (!x || !y) return PERF_ERR_NULL;
    if (!dtype_ok(x_dt) || !dtype_ok(y_dt)) return PERF_ERR_DTYPE;
    if (rows < 1 || cols < 1 || ldx < cols || (axis != 0 && axis != 1)) return PERF_ERR_SHAPE;
    const int64_t need = perf_reduce_mean_workspace_bytes(rows, cols, axis, x_dt);
    if (need < 0) return PERF_ERR_SHAPE;
    if (need > 0 && !workspace) return PERF_ERR_NULL;
    if (need > 0 && !aligned(workspace, 4)) return PERF_ERR_ALIGN;
    const int E = x_dt == PERF_F32 ? 4 : 8;
    // the two-stage path needs 16-byte accesses; everything else is the plain entry point's work
    if (need == 0 || ldx % E != 0 || !aligned(x, 16))
        return perf_reduce_mean(x, y, rows, cols, ldx, axis, x_dt, y_dt, stream);
    if (rows > (INT64_MAX / 4) / ldx) return PERF_ERR_SHAPE;
    if (!aligned(y, dtype_size(y_dt))) return PERF_ERR_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    float *ws = static_cast<float *>(workspace);
    if (x_dt == PERF_F32) {
        if (y_dt == PERF_F32) launch_colmean_ws<float, float>(x, y, ws, rows, cols, ldx, st);
        else launch_colmean_ws<float, uint16_t>(x, y, ws, rows, cols, ldx, st);
    } else {
        if (y_dt == PERF_F32) launch_colmean_ws<uint16_t, float>(x, y, ws, rows, cols, ldx, st);
        else launch_colmean_ws<uint16_t, uint16_t>(x, y, ws, rows, cols, ldx, st);
    }
    return launch_status();
}

extern "C" perf_status perf_eltwise(perf_eltwise_op op, const void *a, const void *b, void *y, int64_t n, perf_dtype dt,
                                    perf_stream stream)
{
    using namespace perf;
    if (op != PERF_ADD && op != PERF_MUL && op != PERF_RELU) return PERF_ERR_UNSUPPORTED;
    if (!a || !y || (op != PERF_RELU && !b)) return PERF_ERR_NULL;
    if (!dtype_ok(dt)) return PERF_ERR_DTYPE;
    if (n < 0) return PERF_ERR_SHAPE;
    if (!aligned(a, dtype_size(dt)) || !aligned(y, dtype_size(dt)) || (op != PERF_RELU && !aligned(b, dtype_size(dt))))
        return PERF_ERR_ALIGN;
    if (n == 0) return PERF_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    return dt == PERF_F32 ? dispatch_eltwise<float>(op, a, b, y, n, st) : dispatch_eltwise<uint16_t>(op, a, b, y, n, st);
}
