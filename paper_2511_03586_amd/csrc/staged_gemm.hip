// perf_gemm beyond the direct global->LDS kernels: other layouts, fp32 operands, any extent, leading
// dimension and alignment, on the staged contraction of staged.h.  (Calls with few tiles mostly run waves_gemm.hip.)
#include <atomic>
#include "staged.h"

namespace perf {

template <typename ASrc, typename BSrc, typename T, typename CT, int TM, int TN, int WM, int WN, int KG, int D>
static perf_status launch(const GemmArgs &g, typename ASrc::Args aa, typename BSrc::Args ba)
{
    using Shape = StagedShape<T, TM, TN, WM, WN, KG>;
    const int tiles_m = (int)((g.M + Shape::BM - 1) / Shape::BM), tiles_n = (int)((g.N + Shape::BN - 1) / Shape::BN);
    auto kern = staged_kernel<ASrc, BSrc, T, CT, TM, TN, WM, WN, KG, D>;
    static std::atomic<bool> attr_done{false};  // raising the dynamic-LDS cap is a per-function, idempotent setting
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, Shape::kLds) !=
            hipSuccess)
            return PERF_ERR_LAUNCH;
        attr_done = true;
    }
    // grid.y carries the batch index; batches beyond the grid limit take further launches
    for (int64_t b0 = 0; b0 < g.batch; b0 += kMaxGridYZ) {
        const unsigned gy = (unsigned)(g.batch - b0 < kMaxGridYZ ? g.batch - b0 : kMaxGridYZ);
        aa.p = (const T *)g.A + b0 * g.strideA;
        ba.p = (const T *)g.B + b0 * g.strideB;
        hipLaunchKernelGGL(kern, dim3((unsigned)((int64_t)tiles_m * tiles_n), gy), dim3(Shape::kThreads * KG), Shape::kLds, g.st, aa,
                           ba, (CT *)g.C + b0 * g.strideC, g.M, g.N, g.K, g.ldc, g.strideC, g.alpha, tiles_m, tiles_n);
    }
    return launch_status();
}

template <typename T, typename CT, int TM, int TN, int WM, int WN, int KG, int D>
static perf_status launch_layouts(const GemmArgs &g)
{
    constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN, kThreads = 64 * WM * WN;
    using AK = KRows<T, BM, kThreads, D>;
    using AR = RRows<T, BM, kThreads, D>;
    using BKr = KRows<T, BN, kThreads, D>;
    using BR = RRows<T, BN, kThreads, D>;
    const DenseArgs<T> aa{nullptr, g.lda, g.strideA}, ba{nullptr, g.ldb, g.strideB};
    if (g.la == PERF_ROW_MAJOR)
        return g.lb == PERF_COL_MAJOR ? launch<AK, BKr, T, CT, TM, TN, WM, WN, KG, D>(g, aa, ba)
                                      : launch<AK, BR, T, CT, TM, TN, WM, WN, KG, D>(g, aa, ba);
    return g.lb == PERF_COL_MAJOR ? launch<AR, BKr, T, CT, TM, TN, WM, WN, KG, D>(g, aa, ba)
                                  : launch<AR, BR, T, CT, TM, TN, WM, WN, KG, D>(g, aa, ba);
}

// An operand's contiguous extent is shorter than its 16-byte loads: element loads for it, and for the other unless that
// has rows along K (2x4096x4096 with both operands column-major, fp32 179 us against 239).
template <typename T, typename CT>
static perf_status launch_any(const GemmArgs &g)
{
    using R = AnyRows<T, 64, 256, 1>;
    using Rows = KRows<T, 64, 256, 1>;
    const bool ar = g.la == PERF_ROW_MAJOR, br = g.lb == PERF_ROW_MAJOR;
    if (!ar && !br && g.K >= 8)
        return launch<R, Rows, T, CT, 1, 1, 2, 2, 1, 1>(g, typename R::Args{nullptr, 1, g.lda, g.strideA}, {nullptr, g.ldb, g.strideB});
    if (ar && br && g.K >= 8)
        return launch<Rows, R, T, CT, 1, 1, 2, 2, 1, 1>(g, {nullptr, g.lda, g.strideA}, typename R::Args{nullptr, 1, g.ldb, g.strideB});
    return launch<R, R, T, CT, 1, 1, 2, 2, 1, 1>(g, typename R::Args{nullptr, ar ? g.lda : 1, ar ? 1 : g.lda, g.strideA},
                                                 typename R::Args{nullptr, br ? 1 : g.ldb, br ? g.ldb : 1, g.strideB});
}

static int64_t tiles_of(const GemmArgs &g, int64_t bm, int64_t bn) { return ((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn) * g.batch; }

// Tile by size, from a sweep over 40 shapes per type in all layouts (us, this choice against the next best):
//   * 256 x 256 (8 waves of 128 x 64; 128 KiB of LDS) for a chip full of them and a reduction long enough to pay
//     for its start: 2999x5003x2048 72 against 80 with 128 x 128; 120 x (125x357x112) 14.7 against 12.8 without it.
//   * 128 x 128 (4 waves, two workgroups per CU) from 192 such tiles on: 952x3562x489 13.6 against 17.4 with 64 x 64.
//   * 64 x 64, four register sets of loads in flight; with few tiles and a long reduction instead two groups of waves
//     that share the K-steps, where launch_waves_gemm leaves such calls: 960x1000x600 row-major 8.2 against 8.7 (9.0 with four
//     groups), 640x1024x896 7.2 against 8.1 (8.6), 999x901x520 with K contiguous 6.6 against 6.9 (7.5), but 1003x1003x513
//     7.6 against 7.4 (8.6), 16 x (256x256x512) 7.2 against 7.1 (8.3); one register set up to K = 64, where the loads for steps that do not exist cost more than the
//     latency they hide (1000x1000x20 6.2 against 5.6, 100x100x36 5.5 against 4.9).
template <typename CT>
static perf_status launch_bf16(const GemmArgs &g, bool big_ok)
{
    if (big_ok && g.K >= 512 && tiles_of(g, 256, 256) >= 192) return launch_layouts<uint16_t, CT, 4, 2, 2, 4, 1, 1>(g);
    if (big_ok && tiles_of(g, 128, 128) >= 192) return launch_layouts<uint16_t, CT, 2, 2, 2, 2, 1, 2>(g);
    if (g.K >= 512 && tiles_of(g, 64, 64) <= 256) return launch_layouts<uint16_t, CT, 1, 1, 2, 2, 2, 2>(g);
    if (g.K <= 64) return launch_layouts<uint16_t, CT, 1, 1, 2, 2, 1, 1>(g);
    return launch_layouts<uint16_t, CT, 1, 1, 2, 2, 1, 4>(g);
}

// fp32: the 256 x 128 tile (8 waves of 64 x 64, 144 KiB of LDS for two stages of three planes) from 128 of them on
// (2696x1608x2139 128 us against 141 with 64 x 64), if they are full (128 x (33x65x36) 11.9 against 6.9 with 64 x 64) or half
// full and the reduction is not short (256 x (128x128x160) 19.4 against 27.8, but x8 9.8 against 9.5), and of 256 on for
// less than a K-step (32 x (512x512x8) 12.6 against 15.0, 2000x2000x16 10.7 against 10.2); else 64 x 64.  128 x 64 was
// never ahead.  One register set up to K = 96 (1000x1000x20 7.1 against 6.3, 512x512x96 6.5 against 5.9).
static perf_status launch_f32(const GemmArgs &g, bool big_ok)
{
    const int64_t big = tiles_of(g, 256, 128), small = tiles_of(g, 64, 64);
    const bool full = 8 * big <= small * 3 / 2, half = 8 * big <= small * 2;
    if (big_ok && big >= 128 && ((full && (big >= 256 || g.K >= 32)) || (half && g.K >= 64)))
        return launch_layouts<float, float, 2, 2, 4, 2, 1, 1>(g);
    if (g.K <= 96) return launch_layouts<float, float, 1, 1, 2, 2, 1, 1>(g);
    return launch_layouts<float, float, 1, 1, 2, 2, 1, 4>(g);
}

perf_status launch_staged_gemm(const GemmArgs &g, int ab_dt, int c_dt)
{
    // (the grid limits of the 64- and 128-wide tiles, whatever tile runs)
    const int64_t edge = tiles_of(g, 128, 128) >= 256 ? 128 : 64;
    if ((g.M + edge - 1) / edge > kMaxGridX || (g.N + edge - 1) / edge > kMaxGridYZ) return PERF_ERR_UNSUPPORTED;
    if (tiles_of(g, 64, 64) / g.batch > max_blocks(256)) {  // (larger tiles and those with wave groups are fewer threads)
        GemmArgs lo = g, hi = g;
        lo.M = g.M / 512 * 256, hi.M = g.M - lo.M;  // (M is at least 2^13: N fits grid.y)
        hi.A = (const char *)g.A + lo.M * (g.la == PERF_ROW_MAJOR ? g.lda : 1) * dtype_size(ab_dt);
        hi.C = (char *)g.C + lo.M * g.ldc * dtype_size(c_dt);
        const perf_status s = launch_staged_gemm(lo, ab_dt, c_dt);
        return s != PERF_OK ? s : launch_staged_gemm(hi, ab_dt, c_dt);
    }
    // the larger tiles hold 32-bit element offsets
    const int64_t v = ab_dt == PERF_BF16 ? 8 : 4;
    const bool few = (g.la == PERF_ROW_MAJOR ? g.K < 8 : g.M < v) || (g.lb == PERF_COL_MAJOR ? g.K < 8 : g.N < v);
    if (few) {
        if (ab_dt == PERF_F32) return launch_any<float, float>(g);
        return c_dt == PERF_F32 ? launch_any<uint16_t, float>(g) : launch_any<uint16_t, uint16_t>(g);
    }
    const bool big_ok = g.lda <= (1 << 21) && g.ldb <= (1 << 21);
    if (ab_dt == PERF_F32) return launch_f32(g, big_ok);
    return c_dt == PERF_F32 ? launch_bf16<float>(g, big_ok) : launch_bf16<uint16_t>(g, big_ok);
}

}  // namespace perf
