// Convolution as an implicit GEMM on the contraction of kwaves.h ("conv" rows of the operator table, Section 4.3 of the
// paper): fp32 operands, and bf16 where the output has few tiles.
#include <atomic>
#include "kwaves.h"

namespace perf {

template <typename T, typename CT, int TM, int TN, int W>
static perf_status launch(const StagedConv &c)
{
    using ASrc = WaveConv<T, TM>;
    using BSrc = WaveRows<T, TN>;
    using Shape = WavesShape<T, TM, TN, W, ASrc, BSrc>;
    const int64_t M = (int64_t)c.N * c.P * c.Q, K = (int64_t)c.R * c.S * c.C;
    const int tiles_m = (int)((M + Shape::BM - 1) / Shape::BM), tiles_n = (c.K + Shape::BN - 1) / Shape::BN;
    auto kern = waves_kernel<ASrc, BSrc, T, CT, TM, TN, W>;
    static std::atomic<bool> attr_done{false};  // raising the dynamic-LDS cap is a per-function, idempotent setting
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, Shape::kLds) !=
            hipSuccess)
            return PERF_ERR_LAUNCH;
        attr_done = true;
    }
    uint32_t tap_rows = 0;
    for (int r = 0; r < c.R; ++r) tap_rows |= 1u << (r * c.S);
    const typename ASrc::Args aa{{(const T *)c.x, c.H, c.W, c.C, c.S, c.sh, c.sw, c.ph, c.pw, c.P, c.Q,
                                  div_magic(c.C), div_magic(c.S), div_magic((int64_t)c.P * c.Q), div_magic(c.Q)},
                                 (uint32_t)((int64_t)c.N * c.H * c.W * c.C * sizeof(T)), tap_rows, c.R};
    hipLaunchKernelGGL(kern, dim3((unsigned)((int64_t)tiles_m * tiles_n)), dim3(Shape::kThreads), Shape::kLds, c.st, aa,
                       DenseArgs<T>{(const T *)c.w, K, 0}, (CT *)c.y, M, (int64_t)c.K, K, (int64_t)c.K, (int64_t)0, 1.0f, tiles_m, tiles_n);
    return launch_status();
}

static int64_t tiles_of(const StagedConv &c, int64_t bm, int64_t bn)
{
    return (((int64_t)c.N * c.P * c.Q + bm - 1) / bm) * ((c.K + bn - 1) / bn);
}

// Tile (32 TM pixels x 32 TN channels) and waves by size, from a sweep over 90 shapes (us, this choice against the staged
// kernel or, for bf16 on whole 32-channel steps (`direct`), the convolution's own main loop):
//   * fp32: 32 x 32 with 8 waves up to 256 tiles (11x16x16x64 -> 64 5x5 11.2 against 26.1), 64 x 32 up to 512 of 32 x 32 (4x81x16x96
//     -> 96 11.0 against 17.9; short reductions 32 x 32 with 4 waves, 16x32x64x16 -> 64 at stride 2 5.6 against 7.7); in one
//     round of 64 x 64 these if the reduction is long (1x208x16x128 -> 256 19.4 against 22.2), else 32 x 32 (5x32x36x64 -> 128
//     11.7 against 13.3), from 288 on (1x1 128 -> 64 6.0 against 5.3) and
//     to 768 of them (6x22x120x64 -> 256 at stride 2 15.8 against 15.1).  Where 64 channels would waste half a tile and more of
//     work is left to win: 64 x 32 in any number (7x16x160x128 -> 96 5x5 99 against 142, 28x160x58x64 -> 32 30.5 against
//     37.6); else 64 x 64 up to two rounds for long reductions (16x24x87x48 -> 64 5x5 36.2 against 40.4; 576 is even).
//   * bf16: 32 x 32 in one round of 64 x 64 (3x208x16x256 -> 32 6.6 against 12.7, 15x16x33x128 -> 96 7.8 against 10.0); 64 x 64
//     with 8 waves for 2000 and more (3x184x20x256 -> 64 5x5 21.8 against 26.8); up to 400 tiles 64 x 64 with 4 waves from 2000 on
//     (6x37x112x128 -> 64 5x5 22.5 against 26.4).  The main loop is ahead or level below 800 (1x16x96x64 -> 128 4.2 against
//     4.3, 8x96x22x64 -> 64 6.2 against 7.0), with 257 to 700 tiles of 32 x 32 below 432 (5x83x32x128 -> 64 1x1 3.6 against 4.6,
//     but 8x64x16x64 -> 64 5.9 against 5.1); the staged kernel below 400.
//     Where 64 channels would waste half a tile: 32 outputs from 576 on 32 x 32 up to 768 tiles (4x64x80x128 -> 32 8.5 against
//     11.4), 64 x 32 up to 4096 (12x21x80x256 -> 32 5x5 26.7 against 47.4, 16x50x60x96 -> 32 11.1 against 12.9, 32x64x64x64 ->
//     32 18.8 against 19.9); more outputs from 2000 on (6x64x192x256 -> 96 at stride 2 23.6 against 27.5, but 8x50x60x128 -> 96
//     17.5 against 15.5).  Channels that the main loop cannot take, 32 outputs: 7x64x120x48 -> 32 9.7 against 14.2.
struct WavesChoice {
    int tm, tn, waves;
};
static WavesChoice choose(const StagedConv &c, int xw_dt, bool direct)
{
    const int64_t t32 = tiles_of(c, 32, 32), t64 = tiles_of(c, 64, 64), k = (int64_t)c.R * c.S * c.C;
    const bool narrow = (c.K + 31) / 32 % 2 == 1;  // the last 64 channels are half a tile
    if (xw_dt == PERF_F32) {
        if (t32 <= 256) return {1, 1, 8};
        if (t32 <= 512) return k >= 400 ? WavesChoice{2, 1, 8} : WavesChoice{1, 1, 4};
        if (narrow && k >= 576) return {2, 1, 4};
        if (t64 <= 256 && k >= (t32 > 768 ? 768 : 1024)) return {2, 2, 8};
        if (t64 <= 256 && k >= 288 && t32 <= 768) return {1, 1, 4};
        if (narrow && k >= 144 && t32 <= 1200) return {1, 1, 4};
        if (t64 <= 512 && k >= 1024) return {2, 2, 4};
        return {0, 0, 0};
    }
    if (k < (!direct ? 400 : t32 > 256 && t32 <= 700 ? 432 : 800)) return {0, 0, 0};
    if (t32 <= 256) return {1, 1, k >= 1024 ? 8 : 4};
    if (c.K <= 32 && k >= 576 && t32 <= 4096) return t32 <= 768 ? WavesChoice{1, 1, 4} : WavesChoice{2, 1, 4};
    if (t64 <= 256) return t64 > 128 && k >= 2000 ? WavesChoice{2, 2, 8} : WavesChoice{1, 1, 4};
    if (narrow && t64 <= 640 && k >= 2000) return {2, 1, 4};
    if (t64 <= 400 && k >= 2000) return {2, 2, 4};
    if (!direct && c.K <= 32 && t32 <= 2048) return {1, 1, 4};
    return {0, 0, 0};
}

template <typename T, typename CT>
static perf_status launch_typed(const StagedConv &c, WavesChoice w)
{
    if (w.tm == 2 && w.tn == 2) return w.waves == 8 ? launch<T, CT, 2, 2, 8>(c) : launch<T, CT, 2, 2, 4>(c);
    if constexpr (sizeof(T) == 4)
        if (w.tm == 2 && w.waves == 8) return launch<T, CT, 2, 1, 8>(c);
    if (w.tm == 2) return launch<T, CT, 2, 1, 4>(c);
    return w.waves == 8 ? launch<T, CT, 1, 1, 8>(c) : launch<T, CT, 1, 1, 4>(c);
}

bool launch_waves_conv(const StagedConv &c, int xw_dt, int y_dt, bool direct, perf_status *status)
{
    // (a K-step at least; chunks of 16 bytes inside a tap; taps as bits; 31-bit byte offsets in x, on whole words, and 32-bit
    // ones in 64 rows of w)
    const int64_t size = dtype_size(xw_dt), k = (int64_t)c.R * c.S * c.C;
    if (k * size < 128 || c.C * size % 16 != 0 || (int64_t)c.R * c.S > 31 || k > (1 << 24) - 64 ||
        (int64_t)c.N * c.H * c.W * c.C * size >= (int64_t(1) << 31) || !aligned(c.x, 4))
        return false;
    // (offsets of taps outside the image, too, and tile numbers)
    if (((int64_t)c.N * c.H + c.R + c.ph) * (c.W + c.S + c.pw) > (int64_t(1) << 31) / (c.C * size) || tiles_of(c, 32, 32) > max_blocks(512))
        return false;
    const WavesChoice w = choose(c, xw_dt, direct);
    if (w.tm == 0) return false;
    if (xw_dt == PERF_BF16)
        *status = y_dt == PERF_F32 ? launch_typed<uint16_t, float>(c, w) : launch_typed<uint16_t, uint16_t>(c, w);
    else
        *status = y_dt == PERF_F32 ? launch_typed<float, float>(c, w) : launch_typed<float, uint16_t>(c, w);
    return true;
}

}  // namespace perf
