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

// Tile (32 TM x 32 TN) and waves by size, from sweeps over some 400 shapes per type in all layouts, single and batched, regular
// and ragged (us, this choice against the staged kernel or, where `direct`, the direct one; [other choices]).  "Rounds" are of
// one workgroup per CU; `whole`: the staged kernel's rounds have no edges to mind, K in whole steps and blocks of 16 bytes.
//   * up to 256 tiles of 32 x 32 these: fp32 with 8 waves (640x24x1920 11.0 against 28, 896x235x3200 19.8 against 42, 80x384x208
//     x4 4.3 against 9.3); bf16 with 8 from K = 1024 on, else 4 (63x208x3673 13.0 against 21.4, 256x64x448 x5 4.0 against 5.8).
//     Where the direct kernel can, from K = 512 on (512x512x512 3.4 against 3.8, [8 waves 3.8]; K = 384 3.4 against 3.4).
//   * bf16 up to 512 such tiles: two of them per wave, along an operand with K strided, whose rows are loaded in pairs, along A if
//     both have (160x2325x968 6.4 against 9.1 [32 x 32 7.9]), unless that has one tile of rows.  32 x 32 for one K-step
//     (whole ones are the staged kernel's: 512x64x64 x16 3.5 against 3.7) and, row-major, below K = 512 (geometric means over
//     six shapes 0.85 [pairs 0.92] at 128, 0.93 [0.97] at 256, but 0.93 [0.92] at 512).
//   * in one round of 64 x 64:
//       bf16, up to two K-steps: 32 x 32 with 2 waves (1024x960x64 3.67 against 3.77 [4 waves 3.88], 999x901x100 4.4 against
//         6.1); fp32 up to three (1024x1024x64 4.6 to 4.7 against 4.7 to 5.0 [4 waves 5.0]), with K contiguous in both to four.
//       bf16 above, B with K strided in A too: pairs to K = 383 (1024x1024x256 4.8 against 5.0 [32 x 32 5.6]), then 64 x 64 with
//         8 waves (1024x1024x384 5.7 against 6.1 [pairs 5.8]); B with K contiguous: pairs to 767 (1024x1024x512 5.75 against 5.9
//         [64 x 64 6.2]; geometric mean over eight at 768 0.73 [0.73]), then these.
//       bf16 row-major: 32 x 32 with 4 below 256 (999x901x200 5.4 against 6.9; at 256 1024x1024 5.4 against 4.8, but 999x901,
//         not whole, 0.89), 64 x 64 with 8 from 1024 on but for single products of whole steps (1024x1024x1024 7.8 against 7.2;
//         705x641x1030 0.5).  In between the staged kernel (768x768x512 4 % ahead).
//       bf16, K contiguous in both: 32 x 32 with 4 to 264 (999x901x200 4.7 against 5.8), 64 x 64 with 8 from 2048 on (geometric
//         mean 0.93; 2488x256x1368 10.7 against 10.2), direct or not: 1024x1024x4096 16.8 against 19.1, but K = 2048 even.
//       fp32: 64 x 64 with 8 waves if they fill half of the chip and K is 512 and more (768x1024x1024 row-major 16.8 against 19.4),
//         but not one-tile matrices with K contiguous in both (64x64x1024 x256 25.1 against 25.3 [27.3]); else 32 x 32 with 4
//         (736x728x144 5.9 against 9.1).
//   * beyond that, to about two and a half rounds, two workgroups per CU.  bf16, not row-major, not one whole K-step (2048x1024x64
//     4.1 against 4.5): pairs, where B has K strided with 2 waves to K = 192 (1280x1280x128 5.1 against 5.8 [4 waves 6.2]), with 4
//     to 511 (448x2653x224 6.0 against 8.1); where not, with 2 to 511 (1280x1280x384 0.91 [1.02] in the mean), with 4 to 767
//     (2560x512x512 6.8 against 7.5 [64 x 64 7.7]); then 64 x 64 with 4 (3904x496x911 12.2 against 14.9).  From one and a half rounds
//     on the staged kernel has whole ones: B with K strided 193 to 1023 (1280x1280x320 7.0 against 7.9 [7.2]), else 512
//     to 767 (2048x1024x512 7.6 against 7.9);
//     with K contiguous in both 32 x 32 with 2 to K = 80 (865x2187x80 5.8 against 6.1 [pairs 6.7]), not from 81 to 383
//     (1300x1300x100 6.8 against 6.3) or from 1500 on (3936x336x2080 21.6 against 20.5).
//     fp32, not K contiguous in both: 64 x 64 with 4 (3480x376x568 19.0 against 23.5), for more than 512 of them 32 x 32 below
//     K = 256 (2300x1000x160 12.5 against 14.0 [14.5]); not up to K = 96 (1024x2512x96 11.2 against 9.5).
struct WavesChoice {
    int tm, tn, waves;
};
static WavesChoice choose(const GemmArgs &g, int ab_dt, bool direct)
{
    const bool bf16 = ab_dt == PERF_BF16, a_rows = g.la == PERF_ROW_MAJOR, b_rows = g.lb == PERF_ROW_MAJOR;
    const bool rows = a_rows && b_rows, both_k = a_rows && !b_rows;
    const bool whole = g.K % 64 == 0 && (a_rows || g.M % 8 == 0) && (!b_rows || g.N % 8 == 0);
    const int64_t t32 = tiles_of(g, 32, 32), t64 = tiles_of(g, 64, 64), K = g.K;
    const WavesChoice none{0, 0, 0};
    if (bf16) {
        const WavesChoice pairs = rows ? (g.N > 32 ? WavesChoice{1, 2, 4} : WavesChoice{2, 1, 4})
                                       : (g.M > 32 ? WavesChoice{2, 1, 4} : WavesChoice{1, 2, 4});
        if (t32 <= 256) return direct && K < 512 ? none : WavesChoice{1, 1, K >= 1024 ? 8 : 4};
        if (direct) return t64 > 128 && t64 <= 256 && K > 2048 ? WavesChoice{2, 2, 8} : none;
        if (t32 <= 512) {
            if (K <= 64 && whole && !rows) return none;
            return K <= 64 || (rows && K < 512) ? WavesChoice{1, 1, 4} : pairs;
        }
        if (t64 <= 256) {
            if (K <= 128) return {1, 1, 2};
            if (both_k) return K <= 264 ? WavesChoice{1, 1, 4} : K >= 2048 ? WavesChoice{2, 2, 8} : none;
            if (rows) return K < 256 || (K == 256 && !whole) ? WavesChoice{1, 1, 4} : K < 1024 || (whole && g.batch == 1) ? none : WavesChoice{2, 2, 8};
            return K < (b_rows ? 384 : 768) ? WavesChoice{2, 1, 4} : WavesChoice{2, 2, 8};
        }
        if (t64 > 512 || rows) return none;
        if (both_k) return K <= 80 ? WavesChoice{1, 1, 2} : K < 384 || K >= 1500 ? none : K < 512 ? WavesChoice{2, 1, 4} : WavesChoice{2, 2, 4};
        if (whole && (K <= 64 || (t64 > 384 && (b_rows ? K > 192 && K < 1024 : K >= 512 && K < 768)))) return none;
        return K <= (b_rows ? 192 : 511) ? WavesChoice{2, 1, 2} : K < (b_rows ? 512 : 768) ? WavesChoice{2, 1, 4} : WavesChoice{2, 2, 4};
    }
    if (t32 <= 256) return {1, 1, 8};
    if (t64 <= 256) {
        if (t64 > 128 && K >= 512 && !(both_k && g.M <= 64 && g.N <= 64)) return {2, 2, 8};
        return {1, 1, t32 > 512 && K <= (both_k ? 128 : 96) ? 2 : 4};
    }
    if (t64 <= 640 && !both_k && K > 96) return t64 > 512 && K < 256 ? WavesChoice{1, 1, 4} : WavesChoice{2, 2, 4};
    return none;
}

template <typename CT>
static perf_status launch_bf16(const GemmArgs &g, WavesChoice c)
{
    if (c.tm == 2 && c.tn == 2) return c.waves == 8 ? launch_layouts<uint16_t, CT, 2, 2, 8>(g) : launch_layouts<uint16_t, CT, 2, 2, 4>(g);
    if (c.tm == 2) return c.waves == 4 ? launch_layouts<uint16_t, CT, 2, 1, 4>(g) : launch_layouts<uint16_t, CT, 2, 1, 2>(g);
    if (c.tn == 2) return launch_layouts<uint16_t, CT, 1, 2, 4>(g);
    if (c.waves == 2) return launch_layouts<uint16_t, CT, 1, 1, 2>(g);
    return c.waves == 8 ? launch_layouts<uint16_t, CT, 1, 1, 8>(g) : launch_layouts<uint16_t, CT, 1, 1, 4>(g);
}
static perf_status launch_f32(const GemmArgs &g, WavesChoice c)
{
    if (c.tm == 2) return c.waves == 8 ? launch_layouts<float, float, 2, 2, 8>(g) : launch_layouts<float, float, 2, 2, 4>(g);
    if (c.waves == 2) return launch_layouts<float, float, 1, 1, 2>(g);
    return c.waves == 8 ? launch_layouts<float, float, 1, 1, 8>(g) : launch_layouts<float, float, 1, 1, 4>(g);
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
    } else {
        *status = launch_f32(g, c);
    }
    return true;
}

}  // namespace perf
