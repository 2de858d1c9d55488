// perf_gemm with fewer output tiles than the chip has room for, on the contraction of kwaves.h.
#include <atomic>
#include "kwaves.h"

namespace perf {

template <typename ASrc, typename BSrc, typename T, typename CT, int TM, int TN, int W>
static perf_status launch(const GemmArgs &g, const typename ASrc::Args &aa, const typename BSrc::Args &ba)
{
    using Shape = WavesShape<T, TM, TN, W, ASrc, BSrc>;
    const int tiles_m = (int)((g.M + Shape::BM - 1) / Shape::BM), tiles_n = (int)((g.N + Shape::BN - 1) / Shape::BN);
    auto kern = waves_kernel<ASrc, BSrc, T, CT, TM, TN, W>;
    static std::atomic<bool> attr_done{false};  // raising the dynamic-LDS cap is a per-function, idempotent setting
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, Shape::kLds) !=
            hipSuccess)
            return PERF_ERR_LAUNCH;
        attr_done = true;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)((int64_t)tiles_m * tiles_n * g.batch)), dim3(Shape::kThreads), Shape::kLds, g.st, aa, ba, (CT *)g.C, g.M,
                       g.N, g.K, g.ldc, g.strideC, g.alpha, tiles_m, tiles_n);
    return launch_status();
}

template <typename T, typename CT, int TM, int TN, int W>
static perf_status launch_layouts(const GemmArgs &g)
{
    const DenseArgs<T> aa{(const T *)g.A, g.lda, g.strideA}, ba{(const T *)g.B, g.ldb, g.strideB};
    if (g.la == PERF_ROW_MAJOR)
        return g.lb == PERF_COL_MAJOR ? launch<WaveRows<T, TM>, WaveRows<T, TN>, T, CT, TM, TN, W>(g, aa, ba)
                                      : launch<WaveRows<T, TM>, WaveCols<T, TN>, T, CT, TM, TN, W>(g, aa, ba);
    return g.lb == PERF_COL_MAJOR ? launch<WaveCols<T, TM>, WaveRows<T, TN>, T, CT, TM, TN, W>(g, aa, ba)
                                  : launch<WaveCols<T, TM>, WaveCols<T, TN>, T, CT, TM, TN, W>(g, aa, ba);
}

static int64_t tiles_of(const GemmArgs &g, int64_t bm, int64_t bn) { return ((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn) * g.batch; }

// Tile (32 TM x 32 TN) and waves by size, from sweeps over 110 shapes per type in all layouts (us, this choice against the
// staged kernel or, where `direct`, the direct one; [other choices]):
//   * 32 x 32 while one round of them leaves CUs idle: fp32 with 8 waves (640x24x1920 11.0 against 28, 896x235x3200 19.8 against
//     42 [64 x 64 41], 80x384x208 x4 4.3 against 9.3); bf16 with 8 from K = 1024 on, else 4 (63x208x3673 13.0 against 21.4,
//     256x64x448 x5 4.0 against 5.8).  The direct kernel is ahead for K under 512 (512x512x384 3.4 against 3.8).
//   * bf16 up to 512 such tiles: two of them per wave, along an operand with K strided, whose rows are loaded in pairs, along A if
//     both have (160x2325x968 6.4 against 9.1 [32 x 32 7.9], 696x720x2232 11.7 against 14.8 [along B 19.2]).
//   * in one round of 64 x 64: these with 8 waves if they fill half of the chip and K is long (768x1024x1024 fp32 row-major
//     16.8 against 19.4, 320x2998x2208 bf16 13.7 against 15.6, 1024x1024x4096 bf16, direct 16.8 against 19.1 but K = 2048 even;
//     bf16 with K contiguous in both from 2048 on: 2488x256x1368 10.7 against 10.2), else 32 x 32 with 4 (736x728x144 fp32 5.9
//     against 9.1, 544x1131x222 bf16 5.2 against 6.5), but not bf16 of middling K (1408x384x528 7.2 against 6.7; row-major
//     960x1000x384 7.4 against 7.0; K contiguous in both 1538x640x349 8.0 against 6.8).
//   * beyond that, to about two and a half rounds, tiles with 4 waves, two workgroups per CU (3480x376x568 fp32 19.0 against 23.5,
//     3904x496x911 bf16 12.2 against 14.9, K under 512 448x2653x224 6.0 against 8.1); fp32 of more than 512 of them 32 x 32 for
//     K under 256 (2300x1000x160 12.5 against 14.0 [14.5]); not for short K (1024x2512x96 fp32 11.2 against 9.5), fp32 with
//     K contiguous in both, row-major bf16 (832x2320x512 10.5 against 9.0) or bf16 with K contiguous in both from 81 to 383
//     (1300x1300x100 6.8 against 6.3) and from 1500 on (3936x336x2080 21.6 against 20.5).
struct WavesChoice {
    int tm, tn, waves;
};
static WavesChoice choose(const GemmArgs &g, int ab_dt, bool direct)
{
    const bool bf16 = ab_dt == PERF_BF16, b_rows = g.lb == PERF_ROW_MAJOR, both_k = g.la == PERF_ROW_MAJOR && !b_rows;
    const int64_t t32 = tiles_of(g, 32, 32), t64 = tiles_of(g, 64, 64);
    if (direct) {
        if (t32 <= 256 && g.K >= 512) return {1, 1, 8};
        if (t64 > 128 && t64 <= 256 && g.K > 2048) return {2, 2, 8};
        return {0, 0, 0};
    }
    if (bf16) {
        const bool a_rows = g.la == PERF_ROW_MAJOR;
        if (t32 <= 256) return {1, 1, g.K >= 1024 ? 8 : 4};
        if (t32 <= 512) return a_rows && b_rows ? WavesChoice{1, 2, 4} : WavesChoice{2, 1, 4};
        const bool rows = a_rows && b_rows;
        if (t64 <= 256 && g.K >= 1024) return g.K < (both_k ? 2048 : b_rows ? 1024 : 1280) ? WavesChoice{0, 0, 0} : WavesChoice{2, 2, 8};
        if (t64 <= 256 && g.K <= (rows ? 256 : both_k ? 264 : 511)) return {1, 1, 4};
        if (t64 <= 256 || t64 > 512 || rows || (both_k && ((g.K > 80 && g.K < 384) || g.K >= 1500))) return {0, 0, 0};
        return g.K >= 512 || (!a_rows && !b_rows && g.K >= 256) ? WavesChoice{2, 2, 4} : WavesChoice{2, 1, 4};
    }
    if (t32 <= 256) return {1, 1, 8};
    if (t64 <= 256) return t64 > 128 && g.K >= 512 ? WavesChoice{2, 2, 8} : WavesChoice{1, 1, 4};
    if (t64 <= 640 && !both_k && g.K > 96) return t64 > 512 && g.K < 256 ? WavesChoice{1, 1, 4} : WavesChoice{2, 2, 4};
    return {0, 0, 0};
}

template <typename CT>
static perf_status launch_bf16(const GemmArgs &g, WavesChoice c)
{
    if (c.tm == 2 && c.tn == 2) return c.waves == 8 ? launch_layouts<uint16_t, CT, 2, 2, 8>(g) : launch_layouts<uint16_t, CT, 2, 2, 4>(g);
    if (c.tm == 2) return launch_layouts<uint16_t, CT, 2, 1, 4>(g);
    if (c.tn == 2) return launch_layouts<uint16_t, CT, 1, 2, 4>(g);
    return c.waves == 8 ? launch_layouts<uint16_t, CT, 1, 1, 8>(g) : launch_layouts<uint16_t, CT, 1, 1, 4>(g);
}

bool launch_waves_gemm(const GemmArgs &g, int ab_dt, int c_dt, bool direct, perf_status *status)
{
    // (a K-step at least; 32-bit byte offsets within 64 rows of fp32)
    constexpr int64_t kMostLd = (1 << 24) - 64;
    if (g.K < (ab_dt == PERF_BF16 ? 64 : 32) || g.K > (1 << 30) || g.lda > kMostLd || g.ldb > kMostLd) return false;
    const WavesChoice c = choose(g, ab_dt, direct);
    if (c.tm == 0) return false;
    if (ab_dt == PERF_BF16) {
        // (pairs of rows of a K-strided operand)
        if ((c.tm == 2 && g.la == PERF_COL_MAJOR && g.M < 2) || (c.tn == 2 && g.lb == PERF_ROW_MAJOR && g.N < 2)) return false;
        *status = c_dt == PERF_F32 ? launch_bf16<float>(g, c) : launch_bf16<uint16_t>(g, c);
    } else if (c.tm == 2) {
        *status = c.waves == 8 ? launch_layouts<float, float, 2, 2, 8>(g) : launch_layouts<float, float, 2, 2, 4>(g);
    } else {
        *status = c.waves == 8 ? launch_layouts<float, float, 1, 1, 8>(g) : launch_layouts<float, float, 1, 1, 4>(g);
    }
    return true;
}

}  // namespace perf
