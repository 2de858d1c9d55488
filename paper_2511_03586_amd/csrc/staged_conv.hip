// Convolution as an implicit GEMM on the staged contraction of staged.h ("conv" rows of the operator table,
// Section 4.3 of the paper): fp32 operands, and channel counts the direct global->LDS kernels do not take.
#include <atomic>
#include "staged.h"

namespace perf {

template <typename ASrc, typename BSrc, typename T, typename CT, int TM, int TN, int WM, int WN, int KG, int D>
static perf_status launch(const StagedConv &c, typename BSrc::Args ba)
{
    using Shape = StagedShape<T, TM, TN, WM, WN, KG>;
    const int64_t M = (int64_t)c.N * c.P * c.Q, K = (int64_t)c.R * c.S * c.C;
    const int tiles_m = (int)((M + Shape::BM - 1) / Shape::BM), tiles_n = (c.K + Shape::BN - 1) / Shape::BN;
    auto kern = staged_kernel<ASrc, BSrc, T, CT, TM, TN, WM, WN, KG, D>;
    static std::atomic<bool> attr_done{false};  // raising the dynamic-LDS cap is a per-function, idempotent setting
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, Shape::kLds) !=
            hipSuccess)
            return PERF_ERR_LAUNCH;
        attr_done = true;
    }
    const typename ASrc::Args aa{(const T *)c.x, c.H, c.W, c.C, c.S, c.sh, c.sw, c.ph, c.pw, c.P, c.Q,
                                 div_magic(c.C), div_magic(c.S), div_magic((int64_t)c.P * c.Q), div_magic(c.Q)};
    hipLaunchKernelGGL(kern, dim3((unsigned)((int64_t)tiles_m * tiles_n), 1), dim3(Shape::kThreads * KG), Shape::kLds, c.st, aa, ba,
                       (CT *)c.y, M, (int64_t)c.K, K, (int64_t)c.K, (int64_t)0, 1.0f, tiles_m, tiles_n);
    return launch_status();
}

// Whole chunks of 8 channels.
template <typename T, typename CT, int TM, int TN, int WM, int WN, int KG, int D>
static perf_status launch_whole(const StagedConv &c)
{
    constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN, kThreads = 64 * WM * WN;
    const int64_t K = (int64_t)c.R * c.S * c.C;
    return launch<ConvRows<T, BM, kThreads, D, true>, KRows<T, BN, kThreads, D>, T, CT, TM, TN, WM, WN, KG, D>(
        c, DenseArgs<T>{(const T *)c.w, K, 0});
}

static int64_t tiles_of(const StagedConv &c, int64_t bm, int64_t bn)
{
    return (((int64_t)c.N * c.P * c.Q + bm - 1) / bm) * ((c.K + bn - 1) / bn);
}

template <typename T, typename CT>
static perf_status launch_typed(const StagedConv &c)
{
    const int64_t K = (int64_t)c.R * c.S * c.C;
    if (c.C % 8 != 0) {
        if (K < 8)
            return launch<ConvRows<T, 64, 256, 1, false>, AnyRows<T, 64, 256, 1>, T, CT, 1, 1, 2, 2, 1, 1>(
                c, typename AnyRows<T, 64, 256, 1>::Args{(const T *)c.w, K, 1, 0});
        return launch<ConvRows<T, 64, 256, 1, false>, KRows<T, 64, 256, 1>, T, CT, 1, 1, 2, 2, 1, 1>(c, DenseArgs<T>{(const T *)c.w, K, 0});
    }
    // Tile by size (us): fp32 takes 128 x 64 from 192 of them on (8x56x56x64->64 21.3 against 22.4 with 64 x 64,
    // 8x28x28x128->256 37.1 against 39.3); two groups of waves where 64 x 64 tiles leave CUs idle and the reduction
    // is long (8x28x28x64->128 fp32 13.3 against 15.6; bf16 with more than 31 taps, 28x28x16->64 x2 7x7 8.1 against 9.3,
    // 28x28x16->64 x8 6x6, 576 long, 7.2 against 7.1).  Larger tiles were never ahead: the pixels' addresses take registers.
    if (sizeof(T) == 4 && K <= (1 << 21) && tiles_of(c, 128, 64) >= 192) return launch_whole<T, CT, 2, 1, 2, 2, 1, 2>(c);
    if constexpr (sizeof(T) == 2)  // ... four groups from 1600 on (8x28x28x64->64 7x7 15.3 against 17.7 with two)
        if (K >= 1600 && tiles_of(c, 64, 64) <= 256) return launch_whole<T, CT, 1, 1, 2, 2, 4, 1>(c);
    if (K >= 512 && tiles_of(c, 64, 64) <= 256) return launch_whole<T, CT, 1, 1, 2, 2, 2, sizeof(T) == 2 ? 2 : 4>(c);
    return launch_whole<T, CT, 1, 1, 2, 2, 1, 4>(c);
}

perf_status launch_staged_conv(const StagedConv &c, int xw_dt, int y_dt)
{
    // (the grid limits of the 64- and 128-wide tiles, whatever tile runs)
    const int64_t edge = tiles_of(c, 128, 128) >= 256 ? 128 : 64;
    if ((c.K + edge - 1) / edge > kMaxGridYZ) return PERF_ERR_UNSUPPORTED;
    if (tiles_of(c, 64, 64) > max_blocks(256) && (c.N > 1 || c.P > 1)) {  // half the images, or half the rows of one
        StagedConv lo = c, hi = c;
        if (c.N > 1) {
            lo.N = c.N / 2, hi.N = c.N - lo.N;
            hi.x = (const char *)c.x + (int64_t)lo.N * c.H * c.W * c.C * dtype_size(xw_dt);
        } else {
            lo.P = c.P / 2, hi.P = c.P - lo.P;
            hi.ph = c.ph - lo.P * c.sh;
        }
        hi.y = (char *)c.y + (int64_t)lo.N * lo.P * c.Q * c.K * dtype_size(y_dt);
        const perf_status s = launch_staged_conv(lo, xw_dt, y_dt);
        return s != PERF_OK ? s : launch_staged_conv(hi, xw_dt, y_dt);
    }
    if (tiles_of(c, 64, 64) > max_blocks(256)) return PERF_ERR_UNSUPPORTED;
    if (xw_dt == PERF_BF16) return y_dt == PERF_F32 ? launch_typed<uint16_t, float>(c) : launch_typed<uint16_t, uint16_t>(c);
    return y_dt == PERF_F32 ? launch_typed<float, float>(c) : launch_typed<float, uint16_t>(c);
}

}  // namespace perf
