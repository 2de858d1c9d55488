// Contractions with fewer output tiles than the chip has room for ("matmul", "bmm" and "conv" rows of the operator
// table, Section 4.3 of the paper): the waves of a workgroup share one output tile and divide K among themselves.
//
//   C[m][n] = alpha * sum_k A(m, k) * B(k, n)         on v_mfma_f32_32x32x16_bf16
//
// Wave w takes the K-steps w, w + W, w + 2 W, ... (128 bytes of a K-contiguous row each) and meets no barrier until its sum
// is complete; the W sums are added in wave order through LDS.  Nothing is shared on the way, so the waves drift apart and
// one's loads, conversions and LDS traffic run beside another's matrix instructions, where the staged contraction
// (staged.h) with one workgroup per CU passes through these phases one after the other:
// 768x1024x1024 fp32, row-major: 2400 cycles per round there for 768 of matrix instructions.
//   * K-contiguous operand (WaveRows): 8 lanes per row and 16 bytes per lane, so that an instruction reads whole lines
//     (a row per lane, as the matrix instruction wants it, moves 17 bytes per clock and CU from the L2, this form 55);
//     passed through 128-byte LDS rows of the wave's own.
//   * K-strided operand (WaveCols): one element (two for bf16) per lane, straight into the matrix instruction's layout.
//   * fp32 is split into three bf16 after that, in registers (split_pair).  If a value did not split and that can show in a
//     sum, the tile is computed again with scaled operands; if a sum is not finite, on the fp32 matrix instruction, which
//     takes the same registers.
// The order of a sum depends on K and W alone, not on the tile.
#pragma once
#include "staged.h"

namespace perf {

// The sources share an interface: init(); rows(k0): the loads of a K-step that are issued at once; cols(k0, s): those of
// its k-substep s (16 k); park(): to LDS; frag(s, i, bits): the 8 elements of the lane in fragment i of substep s, k = 16 s +
// 8 (lane / 32) .. + 7 of the step, as they lie in memory.  kPairs: rows 2 l and 2 l + 1 of 64 are row l of fragments 2 p
// and 2 p + 1 (else row l of fragment i is row 32 i + l).  kTightRegs: not one more to spare beside this source.

// A wave's LDS accesses execute in program order; this holds the compiler to it where a lane reads what another one wrote, or
// writes what another one has read.
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local"); }

// Lane l's chunk l % 8 of rows lds_row(8 i + l / 8) to LDS; wr: the offset for i = 0.
template <int N>
__device__ __forceinline__ void park_rows(char *lds, int wr, const uint4_t (&raw)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i)  // (8 i rows of LDS on, the swizzle changes in constant bits)
        *reinterpret_cast<uint4_t *>(lds + (wr ^ (((i & 1) ^ (i >> 1)) << 4)) + i * 1024) = raw[i];
}
// The lane's 8 elements of a substep in fragment i; rd: the offset of the first 16 bytes in fragment 0.
template <typename T>
__device__ __forceinline__ void frag_rows(const char *lds, int rd, int i, uint4_t (&out)[sizeof(T) / 2])
{
    const int o = (rd ^ ((2 * i & 7) << 4)) + i * 32 * 128;  // (32 i rows on, the swizzle's bits of chunk XOR 2 i)
    out[0] = *reinterpret_cast<const uint4_t *>(lds + o);
    if constexpr (sizeof(T) == 4) out[1] = *reinterpret_cast<const uint4_t *>(lds + (o ^ 16));
}

// Rows of K-contiguous elements, at least one K-step of them.
template <typename T, int TR>
struct WaveRows {
    static constexpr int R = 32 * TR, kLoads = R / 8, KS = 128 / sizeof(T) / 16, kLds = R * 128;
    static constexpr bool kPairs = false, kTightRegs = false;
    using Args = DenseArgs<T>;
    const T *base;
    uint32_t off[kLoads];  // bytes
    uint4_t raw[kLoads];
    char *lds;
    int wr, rd[KS];

    __device__ __forceinline__ void init(const Args &a, int64_t b, int64_t r0, int64_t rows, int lane, char *mine)
    {
        base = a.p + b * a.stride + r0 * a.ld;
        lds = mine;
        const int last = (int)min((int64_t)R, rows - r0) - 1;
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int row = lds_row<64>(8 * i + lane / 8);  // (a wave writes whole bank lines)
            if (i == 0) wr = stage_offset<64>(row, lane % 8);
            off[i] = (uint32_t)(min(row, last) * a.ld * sizeof(T)) + (lane % 8) * 16;
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) rd[s] = stage_offset<64>(lane & 31, sizeof(T) == 2 ? 2 * s + (lane >> 5) : 4 * s + 2 * (lane >> 5));
    }
    __device__ __forceinline__ void rows(int64_t k0)
    {
        const char *b = reinterpret_cast<const char *>(base + k0);
#pragma unroll
        for (int i = 0; i < kLoads; ++i) raw[i] = load_chunk<true>(reinterpret_cast<const T *>(b + off[i]));
    }
    __device__ __forceinline__ void cols(int64_t, int) {}
    __device__ __forceinline__ void park() { park_rows(lds, wr, raw); }
    template <typename S>
    __device__ __forceinline__ void frag(S s, int i, uint4_t (&out)[sizeof(T) / 2]) const
    {
        frag_rows<T>(lds, rd[s], i, out);
    }
};

// The implicit im2col matrix of a convolution over NHWC x of less than 2^31 bytes, whose 16-byte chunks lie in one of at most
// 31 filter taps each: row = output pixel (n, p, q), k = (r, s, c) with c fastest.  Chunks in the zero padding are read past
// the end of the buffer, which gives zeros.
template <typename T, int TR>
struct WaveConv {
    static constexpr int R = 32 * TR, kLoads = R / 8, V = 16 / sizeof(T), KS = 128 / sizeof(T) / 16, kLds = R * 128;
    static constexpr bool kPairs = false, kTightRegs = true;
    struct Args {
        ConvArgs<T> g;
        uint32_t bytes;     // of x
        uint32_t tap_rows;  // bit r S for every filter row r
        int R;
    };
    ConvArgs<T> g;
    rsrc_t rsrc;
    int off[kLoads];        // under tap (0, 0), channel 0: byte offset (may lie outside x)
    uint32_t taps[kLoads];  // bit r S + s: tap (r, s) lies in the image
    int ch;
    uint4_t raw[kLoads];
    char *lds;
    int wr, rd[KS];

    __device__ __forceinline__ void init(const Args &a, int64_t, int64_t r0, int64_t rows, int lane, char *mine)
    {
        g = a.g;
        rsrc = make_rsrc(g.x, a.bytes);
        lds = mine;
        ch = lane % 8;
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int row = lds_row<64>(8 * i + lane / 8);  // (a wave writes whole bank lines)
            if (i == 0) wr = stage_offset<64>(row, ch);
            const int m = (int)min(r0 + row, rows - 1);
            const int n = div_by(m, g.P * g.Q, g.mPQ), pq = m - n * (g.P * g.Q);
            const int p = div_by(pq, g.Q, g.mQ), q = pq - p * g.Q;
            const int ih = p * g.sh - g.ph, iw = q * g.sw - g.pw;
            off[i] = (int)((((int64_t)n * g.H + ih) * g.W + iw) * g.C * (int)sizeof(T));
            const int r_lo = min(max(-ih, 0), a.R), r_hi = max(min(a.R, g.H - ih), 0), s_lo = min(max(-iw, 0), g.S), s_hi = max(min(g.S, g.W - iw), 0);
            auto low = [](int bits) { return (1u << bits) - 1; };
            taps[i] = (a.tap_rows & low(r_hi * g.S) & ~low(r_lo * g.S)) * (low(s_hi) & ~low(s_lo));
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) rd[s] = stage_offset<64>(lane & 31, sizeof(T) == 2 ? 2 * s + (lane >> 5) : 4 * s + 2 * (lane >> 5));
    }
    __device__ __forceinline__ void rows(int64_t k0)
    {
        const int k = (int)k0 + ch * V, t = div_by(k, g.C, g.mC), c = k - t * g.C, r = div_by(t, g.S, g.mS), s = t - r * g.S;
        const int d = ((r * g.W + s) * g.C + c) * (int)sizeof(T);
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const uint32_t from = taps[i] >> t & 1 ? (uint32_t)(off[i] + d) : kOutOfRange;
            raw[i] = __builtin_bit_cast(uint4_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc, from, 0, 0));
        }
    }
    __device__ __forceinline__ void cols(int64_t, int) {}
    __device__ __forceinline__ void park() { park_rows(lds, wr, raw); }
    template <typename S>
    __device__ __forceinline__ void frag(S s, int i, uint4_t (&out)[sizeof(T) / 2]) const
    {
        frag_rows<T>(lds, rd[s], i, out);
    }
};

// K-strided operand: element (row, k) at p[k * ld + row].
template <typename T, int TR>
struct WaveCols;
template <int TR>
struct WaveCols<float, TR> {
    static constexpr int KS = 2, kLds = 0;
    static constexpr bool kPairs = false, kTightRegs = false;
    using Args = DenseArgs<float>;
    const float *base;
    int64_t ld;
    uint32_t off[TR];  // bytes
    uint32_t raw[KS][TR][8];

    __device__ __forceinline__ void init(const Args &a, int64_t b, int64_t r0, int64_t rows, int lane, char *)
    {
        base = a.p + b * a.stride + r0;
        ld = a.ld;
        const int last = (int)min((int64_t)32 * TR, rows - r0) - 1;
#pragma unroll
        for (int i = 0; i < TR; ++i) off[i] = (uint32_t)((lane >> 5) * 32 * a.ld) + 4 * min(i * 32 + (lane & 31), last);
    }
    __device__ __forceinline__ void rows(int64_t) {}
    __device__ __forceinline__ void cols(int64_t k0, int s)
    {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const char *b = reinterpret_cast<const char *>(base + (k0 + 16 * s + e) * ld);
#pragma unroll
            for (int i = 0; i < TR; ++i) raw[s][i][e] = *reinterpret_cast<const uint32_t *>(b + off[i]);
        }
    }
    __device__ __forceinline__ void park() {}
    template <typename S>
    __device__ __forceinline__ void frag(S s, int i, uint4_t (&out)[2]) const
    {
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e >> 2][e & 3] = raw[s][i][e];
    }
};
// bf16, 64 rows and more: a lane loads two rows at once.
template <int TR>
struct WaveCols<uint16_t, TR> {
    static constexpr int KS = 4, kLds = 0;
    static constexpr bool kPairs = TR > 1, kTightRegs = false;
    static constexpr int P = kPairs ? TR / 2 : 1;
    using Args = DenseArgs<uint16_t>;
    const uint16_t *base;
    int64_t ld;
    uint32_t off[P], sel0[P];  // bytes; which half is the even row
    uint32_t raw[KS][P][8];

    __device__ __forceinline__ void init(const Args &a, int64_t b, int64_t r0, int64_t rows, int lane, char *)
    {
        ld = a.ld;
        // An odd last row is the upper half of the pair that ends with it (alone in its tile it takes its neighbour's last
        // row along: the operand has two).
        const int last = (int)min((int64_t)32 * TR, rows - r0) - 1, back = kPairs && last == 0;
        base = a.p + b * a.stride + r0 - back;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int row = kPairs ? 64 * p + 2 * (lane & 31) : lane & 31, at = min(row, kPairs ? last - 1 : last);
            off[p] = (uint32_t)((lane >> 5) * 16 * a.ld) + 2 * (at + back);
            sel0[p] = row > at ? 0x07060302u : 0x05040100u;
        }
    }
    __device__ __forceinline__ void rows(int64_t) {}
    __device__ __forceinline__ void cols(int64_t k0, int s)
    {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const char *b = reinterpret_cast<const char *>(base + (k0 + 16 * s + e) * ld);
#pragma unroll
            for (int p = 0; p < P; ++p) {
                typedef uint32_t word_at2 __attribute__((aligned(2)));
                if constexpr (kPairs) raw[s][p][e] = *reinterpret_cast<const word_at2 *>(b + off[p]);
                else raw[s][p][e] = *reinterpret_cast<const uint16_t *>(b + off[p]);
            }
        }
    }
    __device__ __forceinline__ void park() {}
    template <typename S>
    __device__ __forceinline__ void frag(S s, int i, uint4_t (&out)[1]) const
    {
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const int p = kPairs ? i / 2 : 0;
            const uint32_t lo = raw[s][p][2 * d], hi = raw[s][p][2 * d + 1];
            out[0][d] = __builtin_amdgcn_perm(hi, lo, kPairs && i % 2 ? 0x07060302u : kPairs ? sel0[p] : 0x05040100u);
        }
    }
};

// The largest magnitude among the fp32 values of a step.
__device__ __forceinline__ float larger(float m, uint32_t bits) { return __builtin_fmaxf(m, __builtin_fabsf(__builtin_bit_cast(float, bits))); }
template <int N>
__device__ __forceinline__ float largest_of(const uint4_t (&raw)[N])
{
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) m = larger(m, raw[i][e]);
    return m;
}
template <int KS, int N>
__device__ __forceinline__ float largest_of(const uint32_t (&raw)[KS][N][8])
{
    float m = 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) m = larger(m, raw[s][i][e]);
    return m;
}

template <typename T, int TM, int TN, int W, typename ASrc, typename BSrc>
struct WavesShape {
    static constexpr int BM = 32 * TM, BN = 32 * TN, kThreads = 64 * W, BK = 128 / sizeof(T);
    static constexpr int kSum = TM * TN * 4096;  // a wave's sum
    static constexpr int kWave = ASrc::kLds + BSrc::kLds > kSum ? ASrc::kLds + BSrc::kLds : kSum;
    static constexpr int kLds = kWave * W + 8 * W;  // (and a flag and a value per wave)
    static_assert(kLds <= 160 * 1024, "LDS of one CU");
    // registers: 256 for 64 x 64 (and all but the smallest fp32 tile), 168 and 128 for the smaller ones (fp32 64 x 64 spills 1 to 4
    // of them if B is WaveRows, 11 if A is WaveConv, which spills 1 at 32 x 32)
    static constexpr int kWavesPerSimd = TM * TN == 1 ? 4 : TM * TN == 2 && sizeof(T) == 2 ? 3 : 2;
};

template <typename ASrc, typename BSrc, typename T, typename CT, int TM, int TN, int W>
__global__ __launch_bounds__(64 * W, (WavesShape<T, TM, TN, W, ASrc, BSrc>::kWavesPerSimd)) void waves_kernel(
    typename ASrc::Args aa, typename BSrc::Args ba, CT *__restrict__ C, int64_t M, int64_t N, int64_t K, int64_t ldc, int64_t strideC,
    float alpha, int tiles_m, int tiles_n)
{
    using Shape = WavesShape<T, TM, TN, W, ASrc, BSrc>;
    constexpr int NP = Split<T>::kPlanes, BK = Shape::BK, BM = Shape::BM, BN = Shape::BN, KS = BK / 16, NV = sizeof(T) / 2;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (an XCD's run goes through the batch: a matrix's panels are read into one L2, not into all of them.  64 x (128x128x384) bf16
    // both K-strided 10.6 us without, 7.2 with)
    const unsigned id = xcd_run(blockIdx.x, gridDim.x), tiles = (unsigned)tiles_m * (unsigned)tiles_n;
    const unsigned batch = gridDim.x == tiles ? 0 : id / tiles;
    int tm, tn;
    band_tile(id - batch * tiles, tiles_m, tiles_n, tm, tn);
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    char *const mine = smem + wave * Shape::kWave;
    ASrc sa;
    BSrc sb;
    sa.init(aa, batch, m0, M, lane, mine);
    sb.init(ba, batch, n0, N, lane, mine + ASrc::kLds);
    // The last step starts early enough to be whole; the k of the step before it that it holds too count as zeros.
    const int steps = (int)((K + BK - 1) / BK), count = steps > wave ? (steps - wave + W - 1) / W : 0;
    auto k_of = [&](int i) { return min((int64_t)(wave + i * W) * BK, K - BK); };  // (past the last: the last)
    WaveTile<TM, TN> t;
    Lost lost_of[ASrc::kTightRegs ? 1 : 2], &lost_a = lost_of[0], &lost_b = lost_of[ASrc::kTightRegs ? 0 : 1];
    // A k-substep: its fragments as they lie in memory (read), as the matrix instruction takes them (convert; EDGE: the first
    // `skip` k of the step are zeros), its products (multiply).
    uint4_t ra[TM][NV], rb[TN][NV];
    auto read = [&](auto s) {
#pragma unroll
        for (int i = 0; i < TM; ++i) sa.frag(s, i, ra[i]);
#pragma unroll
        for (int j = 0; j < TN; ++j) sb.frag(s, j, rb[j]);
    };
    auto mask = [&](auto s, uint4_t (&raw)[NV], int skip) {
        const int k = 16 * s + 8 * (lane >> 5);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if constexpr (NP == 1) raw[0][e >> 1] &= k + e < skip ? (e & 1 ? 0x0000ffffu : 0xffff0000u) : 0xffffffffu;
            else raw[e >> 2][e & 3] = k + e < skip ? 0u : raw[e >> 2][e & 3];
        }
    };
    bf16x8_t pa[2][NP][TM], pb[2][NP][TN];
    auto convert = [&](auto s, auto edge, int skip) {
        auto one = [&](uint4_t (&raw)[NV], auto &planes, int i, Lost &lost) {
            if constexpr (decltype(edge)::value) mask(s, raw, skip);
            if constexpr (NP == 1) {
                planes[0][i] = __builtin_bit_cast(bf16x8_t, raw[0]);
            } else {
                uint4_t out[3];
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    uint32_t o[3];
                    const uint32_t lo = raw[d >> 1][2 * (d & 1)], hi = raw[d >> 1][2 * (d & 1) + 1];
                    split_pair<false>(lo, hi, o, lost, 1.f);
#pragma unroll
                    for (int p = 0; p < 3; ++p) out[p][d] = o[p];
                }
#pragma unroll
                for (int p = 0; p < 3; ++p) planes[p][i] = __builtin_bit_cast(bf16x8_t, out[p]);
            }
        };
#pragma unroll
        for (int i = 0; i < TM; ++i) one(ra[i], pa[s & 1], i, lost_a);
#pragma unroll
        for (int j = 0; j < TN; ++j) one(rb[j], pb[s & 1], j, lost_b);
    };
    auto multiply = [&](auto s) {
        constexpr int c = s & 1;
        if constexpr (NP == 1) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    t.acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pa[c][0][i], pb[c][0][j], t.acc[i][j], 0, 0, 0);
        } else {
            constexpr int kPa[6] = {1, 0, 2, 0, 1, 0}, kPb[6] = {1, 2, 0, 1, 0, 0};  // the small products first
#pragma unroll
            for (int q = 0; q < 6; ++q)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        t.acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pa[c][kPa[q]][i], pb[c][kPb[q]][j], t.acc[i][j], 0, 0, 0);
        }
    };
    // Parks a step; load(): the loads that take its registers.  (The compiler moves none past a fence: beside the convolution's
    // source they go between the writes, 4x28x28x64 -> 128 fp32 8.5 us against 8.75, 768x768x1024 with K contiguous 16.0 behind them
    // against 16.9.)
    auto park = [&](auto &&load) {
        wave_lds_fence();  // (the step before has been read)
        sa.park();
        sb.park();
        if constexpr (ASrc::kTightRegs) load();
        wave_lds_fence();
        if constexpr (!ASrc::kTightRegs) load();
    };
    // A step whose substep 0 is converted: the next substep's fragments are read and converted beside the products of one,
    // and behind the last one's reads the next step (NEXT) takes the LDS and the one after that the registers of its loads.
    auto step = [&](auto next, auto edge, auto next_edge, int i, int skip) {
        constexpr bool kNext = decltype(next)::value;
        unrolled<KS>([&](auto s) {
            constexpr bool kLast = s + 1 == KS;
            if constexpr (kNext) {  // (the registers of a K-strided operand's substep are free when it is converted)
                sa.cols(k_of(i + 1), s);
                sb.cols(k_of(i + 1), s);
            }
            if constexpr (!kLast) {
                read(std::integral_constant<int, s + 1>{});
            } else if constexpr (kNext) {
                park([&]() {
                    sa.rows(k_of(i + 2));
                    sb.rows(k_of(i + 2));
                });
                read(std::integral_constant<int, 0>{});
            }
            __builtin_amdgcn_sched_barrier(0);
            multiply(s);
            if constexpr (!kLast) convert(std::integral_constant<int, s + 1>{}, edge, skip);
            else if constexpr (kNext) convert(std::integral_constant<int, 0>{}, next_edge, skip);
            if constexpr (NP > 1 && (kNext || !kLast)) {
                // (one instruction of the matrix unit takes 32 cycles, the conversions' 2.3 to 4.2 each)
                constexpr int kMfma = 6 * TM * TN, kPer = (48 * (TM + TN) + kMfma - 1) / kMfma;
                unrolled<kMfma>([&](auto) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, kPer, 0);
                });
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    auto start = [&](int64_t k0) {
        sa.rows(k0);
        sb.rows(k0);
        unrolled<KS>([&](auto s) {
            sa.cols(k0, s);
            sb.cols(k0, s);
        });
    };
    const int skip = (int)max((int64_t)0, (int64_t)steps * BK - K);  // of the last step
    const std::true_type yes;
    const std::false_type no;
    t.clear();
    if (count > 0) {
        const bool ends = wave + (count - 1) * W == steps - 1;
        const int cut = ends ? skip : 0;
        start(k_of(0));
        park([&]() {
            sa.rows(k_of(1));
            sb.rows(k_of(1));
        });
        read(std::integral_constant<int, 0>{});
        convert(std::integral_constant<int, 0>{}, yes, count == 1 ? cut : 0);
        int i = 0;
        for (; i + 2 < count; ++i) step(yes, no, no, i, 0);
        if (i + 1 < count) step(yes, no, yes, i, cut);
        step(no, yes, no, 0, cut);
    }
    // The sum again without the overlap, from step `first` on: split once more, the operands times times_a and times_b (SCALED;
    // then every fp32 value fits), or on the fp32 instruction, which takes 2.7 times the cycles (all of A of 768x1024x1024 under
    // 2^-110: 32 us for 36).
    auto sum_again = [&](auto scaled, int first, float times_a, float times_b) {
        constexpr bool kScaled = decltype(scaled)::value;
        t.clear();
        for (int i = first; i < count; ++i) {
            start(k_of(i));
            park([]() {});
            const int cut = wave + i * W == steps - 1 ? skip : 0;
            unrolled<KS>([&](auto s) {
                read(s);
                if constexpr (kScaled) {
                    auto scale = [&](uint4_t (&raw)[NV], float times) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const uint32_t bits = raw[e >> 2][e & 3];
                            raw[e >> 2][e & 3] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(float, bits) * times);
                        }
                    };
#pragma unroll
                    for (int m = 0; m < TM; ++m) scale(ra[m], times_a);
#pragma unroll
                    for (int n = 0; n < TN; ++n) scale(rb[n], times_b);
                    convert(s, yes, cut);
                    multiply(s);
                } else {
#pragma unroll
                    for (int m = 0; m < TM; ++m) mask(s, ra[m], cut);
#pragma unroll
                    for (int n = 0; n < TN; ++n) mask(s, rb[n], cut);
#pragma unroll
                    for (int e = 0; e < 8; ++e)
#pragma unroll
                        for (int m = 0; m < TM; ++m)
#pragma unroll
                            for (int n = 0; n < TN; ++n) {
                                const uint32_t x = ra[m][e >> 2][e & 3], y = rb[n][e >> 2][e & 3];
                                t.acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float, x), __builtin_bit_cast(float, y),
                                                                                  t.acc[m][n], 0, 0, 0);
                            }
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        }
        if constexpr (kScaled) {
            const float back_a = times_a > 1.f ? 0x1p-24f : 1.f, back_b = times_b > 1.f ? 0x1p-24f : 1.f;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) t.acc[i][j][e] *= back_a * back_b;
        }
    };
    // Sums to LDS in quads of rows; quad u of the tile (TM * TN * 4 of them, 64 lanes each) is added and stored by wave u % W.
    auto leave = [&]() {
        wave_lds_fence();  // (the last step has been read)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float4_t *>(mine + (((i * TN + j) * 4 + q) * 64 + lane) * 16) =
                        float4_t{t.acc[i][j][4 * q], t.acc[i][j][4 * q + 1], t.acc[i][j][4 * q + 2], t.acc[i][j][4 * q + 3]};
    };
    // Quad u of the tile's sums.
    auto total = [&](int u) {
        const char *from = smem + (u * 64 + lane) * 16;
        float4_t v = *reinterpret_cast<const float4_t *>(from);
#pragma unroll
        for (int w = 1; w < W; ++w) v += *reinterpret_cast<const float4_t *>(from + w * Shape::kWave);
        return v;
    };
    leave();
    if constexpr (NP > 1) {
        auto not_finite = [&]() {
            float z = 0.f;  // (infinities and NaN make it NaN)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) z = __builtin_fmaf(t.acc[i][j][e], 0.f, z);
            return __any(z != 0.f);
        };
        int *flags = reinterpret_cast<int *>(smem + Shape::kWave * W);
        float *values = reinterpret_cast<float *>(flags + W);
        // Any wave's flags, in all of them (a barrier: the sums are complete behind it).
        auto any_of = [&](int mine) {
            if (lane == 0) flags[wave] = mine;
            __syncthreads();
            int any = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) any |= flags[w];
            return __builtin_amdgcn_readfirstlane(any);
        };
        constexpr int kLostA = 1, kLostB = 2, kNotFinite = 4;
        const int met = any_of((__any(lost_a.any()) ? kLostA : 0) | (__any(lost_b.any()) ? kLostB : 0) | (not_finite() ? kNotFinite : 0));
        if (met) {
            int first = 0;
            asm volatile("" : "+s"(first));  // (what the compiler would keep for this costs the loop above registers)
            bool unit = (met & kNotFinite) != 0, again = unit;
            if (!unit) {
                // A value loses less than 2^-133, so a sum less than 2^-133 K max |other operand|: nothing that shows if
                // every sum is 2^28 times that.  (Probabilities times values: those that underflow stand beside others.
                // A few of them in A of 1024x2048x512: 19 us for 36 with the repeat, none 16.)
                auto largest = [&](const auto &src) {
                    float m = 0.f;
                    for (int i = first; i < count; i += 4)  // (four steps in flight: the loads' latency counts here)
                        unrolled<4>([&](auto u) {
                            auto step_of = src;
                            step_of.rows(k_of(i + u));
                            unrolled<KS>([&](auto s) { step_of.cols(k_of(i + u), s); });
                            m = __builtin_fmaxf(m, largest_of(step_of.raw));
                        });
                    return m;
                };
                float big = met & kLostA ? largest(sb) : 0.f;
                if (met & kLostB) big = __builtin_fmaxf(big, largest(sa));
                big = wave_allreduce(big, OpMax{});
                if (lane == 0) values[wave] = big;
                __syncthreads();
#pragma unroll
                for (int w = 0; w < W; ++w) big = __builtin_fmaxf(big, values[w]);
                const float least = 0x1p-104f * (float)K * big;  // (2^29 times: both operands may have lost)
                bool small = false;
                for (int u = first + wave; u < TM * TN * 4; u += W) {
                    const float4_t v = total(u);
#pragma unroll
                    for (int e = 0; e < 4; ++e) small |= !(__builtin_fabsf(v[e]) >= least);
                }
                again = any_of(__any(small)) != 0;
            }
            if (again) {
                if (!unit) {
                    sum_again(yes, first, met & kLostA ? 0x1p24f : 1.f, met & kLostB ? 0x1p24f : 1.f);
                    __syncthreads();  // (the flags have been read)
                    unit = any_of(not_finite()) != 0;
                }
                if (unit) sum_again(no, first, 1.f, 1.f);
                leave();
                __syncthreads();
            }
        }
    } else {
        __syncthreads();
    }
    const int rows = (int)min((int64_t)BM, M - m0), cols = (int)min((int64_t)BN, N - n0);
    CT *Ct = C + (int64_t)batch * strideC + m0 * ldc + n0;
#pragma unroll
    for (int u0 = 0; u0 < TM * TN * 4; u0 += W) {
        const int u = u0 + wave;
        if (W > 4 * TM * TN && u >= TM * TN * 4) break;
        const float4_t v = total(u);
        const int q = u % 4, i = u / (4 * TN), j = u / 4 % TN, l = 8 * q + 4 * (lane >> 5);
        const int c = BSrc::kPairs ? 64 * (j / 2) + 2 * (lane & 31) + j % 2 : 32 * j + (lane & 31);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int r = ASrc::kPairs ? 64 * (i / 2) + 2 * (l + e) + i % 2 : 32 * i + l + e;
            if (r < rows && c < cols) store_c<CT>(Ct + (int64_t)r * ldc + c, alpha * v[e]);
        }
    }
}

}  // namespace perf
