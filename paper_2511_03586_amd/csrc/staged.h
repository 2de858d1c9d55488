// Contractions whose operands cannot go to LDS as they lie in memory ("matmul", "bmm" and "conv"
// rows of the operator table, Section 4.3 of the paper): layouts with K strided, any extent, leading
// dimension and alignment, fp32 operands, and the implicit im2col matrix of a convolution.
//
//   C[m][n] = alpha * sum_k A(m, k) * B(k, n)         on v_mfma_f32_32x32x16_bf16
//
// The operands pass through registers on their way to LDS, where every operand ends up as rows of
// K-contiguous bf16 (XOR-swizzled 16-byte chunks, as in mfma_tile.h).  What happens on the way:
//   * K-contiguous rows (KRows): 16-byte loads at the element's own alignment.
//   * K-strided operands (RRows: column-major A, row-major B): a thread loads 16 bytes of four
//     consecutive k-rows and transposes the block with byte permutes.
//   * convolution activations (ConvRows): the chunk's filter tap is decoded per step; taps in the
//     zero padding are zeroed.
//   * fp32: every value is split exactly into three bf16 (a = a0 + a1 + a2, each the nearest bf16 to what the ones
//     before leave), and a product is the six MFMAs a0b0, a0b1, a1b0, a1b1, a0b2, a2b0.  |a1| <= 2^-8 and |a2| <= 2^-17
//     of a's power of two, so what is left out is at most 2^-24 of the product, of either sign (by truncation, whose
//     parts share the sign of the value, it was up to 2^-21 and always towards zero).  The fp32 accumulator is
//     rounded 6/16 times per k instead of once with the fp32 matrix instruction, which outweighs that from a few k on
//     (rms error against float64 over sum |a||b|, operands in [-1, 1): K = 1024 1.4e-8 for 2.4e-8, K = 8 1.3e-8 for 2.5e-8,
//     but K = 1 3.3e-8 for 2.5e-8); K < 8 takes the fp32 instruction.
//     bf16 ends at 2^-133, so that a value under 2^-110 may not fit: a workgroup that met one computes its tile again
//     with that operand times 2^24 (TIMES), and then every fp32 value fits.  Next to FLT_MAX (2^104 the second time) a0
//     rounds to infinity: sums that are not finite are computed with the fp32 matrix instruction, straight from memory.
// Pipeline: the values of step s+2 are in flight while step s+1's go from registers to the other
// LDS stage and step s is multiplied; one barrier per step.  KG > 1 splits the K-steps among KG
// groups of waves of the workgroup, whose sums are added through LDS in a fixed order.
#pragma once
#include <type_traits>
#include "host_utils.h"
#include "mfma_tile.h"
#include "row_io.h"

namespace perf {

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(uint16_t v) { return bf16_to_f32(v); }

template <typename T> struct Split;
template <> struct Split<uint16_t> {
    static constexpr int kPlanes = 1, kBK = 64, kVec = 8;  // bf16 planes, K-step, elements per 16 bytes
};
template <> struct Split<float> {
    static constexpr int kPlanes = 3, kBK = 32, kVec = 4;
};

// What a split did not hold, as bits of its last residual: a bf16 is the upper half of an fp32.
struct Lost {
    uint32_t v = 0;
    __device__ __forceinline__ bool any() const { return (v & 0xffffu) != 0; }
};

// One conversion for both values.  (The compiler otherwise converts the upper one a second time to widen it again.)
__device__ __forceinline__ uint32_t pack_once(float lo, float hi)
{
    uint32_t v = pack_bf16(lo, hi);
    asm("" : "+v"(v));
    return v;
}

// Two fp32 values, times a power of two if TIMES, as pairs of bf16: out[p] holds plane p of (lo, hi).  (The subtractions
// are exact.)
template <bool TIMES>
__device__ __forceinline__ void split_pair(uint32_t lo, uint32_t hi, uint32_t (&out)[3], Lost &lost, float times)
{
    float l0 = __builtin_bit_cast(float, lo), h0 = __builtin_bit_cast(float, hi);
    if constexpr (TIMES) {
        l0 *= times;
        h0 *= times;
    }
    out[0] = pack_once(l0, h0);
    const float l1 = l0 - bf16_lo(out[0]), h1 = h0 - bf16_hi(out[0]);
    out[1] = pack_once(l1, h1);
    const uint32_t l2 = __builtin_bit_cast(uint32_t, l1 - bf16_lo(out[1])), h2 = __builtin_bit_cast(uint32_t, h1 - bf16_hi(out[1]));
    out[2] = __builtin_amdgcn_perm(h2, l2, 0x07060302u);
    lost.v |= l2 | h2;
}

// LDS image of an operand: planes of ROWS rows of BK bf16 (128 or 64 bytes).  Within 16 rows the order is
// permuted (lds_row) and the 16-byte chunk c of row r sits at c ^ swz(r), so that both kinds of access fall on all
// 16 slots of a 256-byte bank line: the reads (16 consecutive rows at one chunk, in the lane groups that a
// ds_read_b128 takes at a time) and the transposing writes of a K-strided operand, whose lanes are 8 (bf16) or
// 4 (fp32) rows apart.
template <int BK>
__device__ __forceinline__ int lds_row(int r)  // its own inverse
{
    return BK == 64 ? (r & ~9) | ((r & 1) << 3) | ((r >> 3) & 1)       // bits 0 and 3 exchanged
                    : (r & ~15) | ((r & 3) << 2) | ((r >> 2) & 3);     // bits 1:0 and 3:2 exchanged
}
template <int BK>
__device__ __forceinline__ int stage_offset(int row, int chunk)
{
    const int s = BK == 64 ? (row ^ (row >> 4)) & 7 : (row ^ (row >> 4)) & 3;
    return lds_row<BK>(row) * (2 * BK) + ((chunk ^ s) << 4);
}
// ... of row + STEP, given the offset of a row below STEP (a power of two >= 16): the swizzle is one XOR.
template <int BK>
__device__ __forceinline__ int stage_step(int o, int step)
{
    return (o ^ (((step >> 4) & (BK / 8 - 1)) << 4)) + step * (2 * BK);
}

// A vector (or two) of elements moved down by `sh` >= 0 places, zeros moving in.
template <typename T, int V>
__device__ __forceinline__ void shift_down(uint4_t (&v)[V], int sh)
{
    uint32_t w[4 * V];
#pragma unroll
    for (int d = 0; d < 4 * V; ++d) w[d] = v[d >> 2][d & 3];
    const int words = sizeof(T) == 2 ? sh >> 1 : sh;
    auto by = [&](auto step, bool go) {
#pragma unroll
        for (int d = 0; d < 4 * V; ++d) {
            const uint32_t from = d + step < 4 * V ? w[d + step < 4 * V ? d + step : 0] : 0u;
            w[d] = go ? from : w[d];
        }
    };
    if constexpr (V == 2) by(std::integral_constant<int, 4>{}, (words & 4) != 0);
    by(std::integral_constant<int, 2>{}, (words & 2) != 0);
    by(std::integral_constant<int, 1>{}, (words & 1) != 0);
    by(std::integral_constant<int, 4 * V>{}, words >= 4 * V);
    if constexpr (sizeof(T) == 2) {
        const bool half = (sh & 1) != 0;
#pragma unroll
        for (int d = 0; d < 4 * V; ++d) w[d] = half ? (w[d] >> 16) | (d + 1 < 4 * V ? w[d + 1] << 16 : 0u) : w[d];
    }
#pragma unroll
    for (int d = 0; d < 4 * V; ++d) v[d >> 2][d & 3] = w[d];
}

// Park a chunk of 8 K-contiguous elements at offset `o` of every plane.
template <typename T, int ROWS, bool TIMES>
__device__ __forceinline__ void park_chunk(char *lds, int o, const uint4_t (&r)[8 / Split<T>::kVec], Lost &lost, float times)
{
    if constexpr (Split<T>::kPlanes == 1) {
        *reinterpret_cast<uint4_t *>(lds + o) = r[0];
    } else {
        uint4_t pl[3];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t out[3];
            const uint32_t lo = r[d >> 1][2 * (d & 1)], hi = r[d >> 1][2 * (d & 1) + 1];
            split_pair<TIMES>(lo, hi, out, lost, times);
#pragma unroll
            for (int p = 0; p < 3; ++p) pl[p][d] = out[p];
        }
#pragma unroll
        for (int p = 0; p < 3; ++p) *reinterpret_cast<uint4_t *>(lds + p * (ROWS * 2 * Split<T>::kBK) + o) = pl[p];
    }
}

template <typename T>
struct DenseArgs {
    const T *p;
    int64_t ld, stride;  // leading dimension, distance of the batch's matrices
};

// The operand sources below share an interface: init(), whole() (uniform: no row of the tile needs an
// edge case), fetch<EDGE>(k0, slot) (loads of the K-step at k0 into register set `slot`) and
// park<EDGE, TIMES>(lds, k0, slot).  EDGE = false requires a whole K-step, and whole() where it is parked; past K, EDGE
// fetches stay inside the operand and EDGE parks zeros.  lost, times: see split_pair (fp32).  at(row, k):
// one element of the tile as fp32, zero outside.

// Rows of K-contiguous elements, K >= 8.  An item is one chunk of 8 elements of a row; a chunk that would
// overhang K is loaded from K - 8 on and moved down.
template <typename T, int ROWS, int THREADS, int D>
struct KRows {
    using S = Split<T>;
    using Shallow = KRows<T, ROWS, THREADS, 1>;  // one register set
    static constexpr bool kElements = false;  // loads element by element
    static constexpr int kDepth = D;
    static constexpr int BK = S::kBK, CH = BK / 8, ITEMS = ROWS * CH, PER = ITEMS / THREADS, V = 8 / S::kVec;
    static constexpr int kRowStep = THREADS / CH, kBlock = 1;
    static_assert(ITEMS % THREADS == 0 && kRowStep >= 16, "items divide among the threads, one chunk column per thread");
    using Off = std::conditional_t<(ROWS > 64), uint32_t, int64_t>;
    using Args = DenseArgs<T>;
    const T *base;
    Off off[PER];  // elements from `base`, without the chunk's
    int64_t K;
    int ch, o0, last;
    uint4_t raw[D][PER][V];
    Lost lost;
    float times;

    __device__ __forceinline__ void init(const Args &a, int64_t b, int64_t r0, int64_t rows, int64_t K_, int tid)
    {
        base = a.p + b * a.stride + r0 * a.ld;
        K = K_;
        ch = tid % CH;
        const int row = lds_row<BK>(tid / CH);  // (a wave writes whole bank lines)
        last = (int)min((int64_t)ROWS, rows - r0) - 1;
        o0 = stage_offset<BK>(row, ch);
#pragma unroll
        for (int i = 0; i < PER; ++i) off[i] = (Off)((int64_t)min(row + i * kRowStep, last) * a.ld);
    }
    __device__ __forceinline__ bool whole() const { return true; }
    __device__ __forceinline__ float at(const Args &a, int row, int64_t k) const
    {
        const float v = to_f32(base[min(row, last) * a.ld + min(k, K - 1)]);
        return row <= last && k < K ? v : 0.f;
    }
    template <bool EDGE>
    __device__ __forceinline__ void fetch(int64_t k0, int slot)
    {
        const int64_t ku = EDGE ? min(k0, K - 8) : k0;
        const Off d = EDGE ? (Off)min((int64_t)ch * 8, K - 8 - ku) : (Off)(ch * 8);
        const T *b = base + ku;
#pragma unroll
        for (int i = 0; i < PER; ++i)
#pragma unroll
            for (int v = 0; v < V; ++v) raw[slot][i][v] = load_chunk<true>(b + (Off)(off[i] + d) + v * S::kVec);
    }
    template <bool EDGE, bool TIMES>
    __device__ __forceinline__ void park(char *lds, int64_t k0, int slot)
    {
        if constexpr (EDGE) {
            if (k0 + BK > K) {
                const int sh = (int)max((int64_t)0, k0 + ch * 8 - (K - 8));
#pragma unroll
                for (int i = 0; i < PER; ++i) shift_down<T, V>(raw[slot][i], sh);
            }
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            park_chunk<T, ROWS, TIMES>(lds, stage_step<BK>(o0, i * kRowStep), raw[slot][i], lost, times);
        }
    }
};

// K-strided operand: element (row, k) at p[k * ld + row].  An item is a block of V rows x KB k (V = 8 bf16 or
// 4 fp32 = 16 bytes; KB = 4, or 2 where 4 would leave half the threads idle), transposed on the way to LDS.  A block that would overhang the last row is loaded from V
// rows before the end and moved down, so every load stays inside the tile, which has at least V rows (the operand has
// that many, and a later tile starts early enough to end on a whole block).
template <typename T, int ROWS, int THREADS, int D>
struct RRows {
    using S = Split<T>;
    using Shallow = RRows<T, ROWS, THREADS, 1>;  // one register set
    static constexpr bool kElements = false;  // loads element by element
    static constexpr int kDepth = D;
    static constexpr int BK = S::kBK, V = S::kVec, RB = ROWS / V, KB = RB * BK / THREADS;
    static constexpr int kBlock = V;
    static_assert(KB == 2 || KB == 4, "one block per thread");
    using Off = std::conditional_t<(ROWS > 64), uint32_t, int64_t>;
    using Args = DenseArgs<T>;
    const T *base;
    int64_t ld, K;
    Off off;
    int kq, sh, o0, last;
    bool all;
    uint4_t raw[D][KB];
    Lost lost;
    float times;

    __device__ __forceinline__ void init(const Args &a, int64_t b, int64_t r0, int64_t rows, int64_t K_, int tid)
    {
        ld = a.ld;
        K = K_;
        // 16 row blocks x 4 k-blocks per wave: 256 contiguous bytes of each k-row
        constexpr int L = RB < 16 ? RB : 16;
        const int rb = tid % L + (tid / (L * (BK / KB))) * L;
        kq = (tid / L) % (BK / KB) * KB;
        const int valid = (int)min((int64_t)ROWS, rows - r0), start = min(rb * V, valid - V);
        sh = rb * V < valid ? rb * V - start : 0;  // (a block of rows that are never stored may hold anything)
        all = valid % V == 0;
        last = valid - 1;
        base = a.p + b * a.stride + r0;
        off = (Off)((int64_t)kq * a.ld + start);
        o0 = stage_offset<BK>(rb * V, kq >> 3) + (kq & 7) * 2;
    }
    __device__ __forceinline__ bool whole() const { return all; }
    __device__ __forceinline__ float at(const Args &, int row, int64_t k) const
    {
        const float v = to_f32(base[min(k, K - 1) * ld + min(row, last)]);
        return row <= last && k < K ? v : 0.f;
    }
    template <bool EDGE>
    __device__ __forceinline__ void fetch(int64_t k0, int slot)
    {
        if constexpr (EDGE) {
            const Off start = off - (Off)((int64_t)kq * ld);
#pragma unroll
            for (int u = 0; u < KB; ++u) raw[slot][u] = load_chunk<true>(base + min(k0 + kq + u, K - 1) * ld + start);
        } else {
            const T *b = base + k0 * ld;
#pragma unroll
            for (int u = 0; u < KB; ++u) raw[slot][u] = load_chunk<true>(b + u * ld + off);
        }
    }
    template <bool EDGE, bool TIMES>
    __device__ __forceinline__ void park(char *lds, int64_t k0, int slot)
    {
        if constexpr (EDGE) {
            if (!all || k0 + BK > K) {
#pragma unroll
                for (int u = 0; u < KB; ++u) {
                    uint4_t v[1] = {raw[slot][u]};
                    shift_down<T, 1>(v, k0 + kq + u < K ? sh : V);
                    raw[slot][u] = v[0];
                }
            }
        }
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const int o = (o0 ^ (e << 4)) + (BK == 64 ? (e & 1) * 8 + (e >> 1) * 2 : e * 4) * (2 * BK);  // row rb * V + e
            uint32_t pair[KB / 2][3];  // the k-pairs of row e, per plane
#pragma unroll
            for (int h = 0; h < KB / 2; ++h) {
                if constexpr (S::kPlanes == 1) {
                    const uint32_t lo = raw[slot][2 * h][e >> 1], hi = raw[slot][2 * h + 1][e >> 1];
                    pair[h][0] = __builtin_amdgcn_perm(hi, lo, (e & 1) ? 0x07060302u : 0x05040100u);
                } else {
                    const uint32_t lo = raw[slot][2 * h][e], hi = raw[slot][2 * h + 1][e];
                    split_pair<TIMES>(lo, hi, pair[h], lost, times);
                }
            }
#pragma unroll
            for (int p = 0; p < S::kPlanes; ++p) {
                char *dst = lds + p * (ROWS * 2 * BK) + o;
                if constexpr (KB == 4) *reinterpret_cast<uint2_t *>(dst) = uint2_t{pair[0][p], pair[1][p]};
                else *reinterpret_cast<uint32_t *>(dst) = pair[0][p];
            }
        }
    }
};

// Any strides, any extent (operands too small for 16-byte loads): element loads.
template <typename T, int ROWS, int THREADS, int D>
struct AnyRows {
    using S = Split<T>;
    using Shallow = AnyRows<T, ROWS, THREADS, 1>;  // one register set
    static constexpr bool kElements = true;  // loads element by element
    static constexpr int kDepth = D;
    static constexpr int BK = S::kBK, CH = BK / 8, PER = ROWS * CH / THREADS, V = 8 / S::kVec, kRowStep = THREADS / CH, kBlock = 1;
    struct Args {
        const T *p;
        int64_t s_row, s_k, stride;
    };
    Args g;
    int64_t K;
    int row, ch, last;
    uint4_t raw[D][PER][V];
    Lost lost;
    float times;

    __device__ __forceinline__ void init(const Args &a, int64_t b, int64_t r0, int64_t rows, int64_t K_, int tid)
    {
        g = a;
        g.p += b * a.stride + r0 * a.s_row;
        K = K_;
        ch = tid % CH;
        row = tid / CH;
        last = (int)min((int64_t)ROWS, rows - r0) - 1;
    }
    __device__ __forceinline__ bool whole() const { return false; }
    __device__ __forceinline__ float at(const Args &, int r, int64_t k) const
    {
        const float v = to_f32(g.p[min(k, K - 1) * g.s_k + min(r, last) * g.s_row]);
        return r <= last && k < K ? v : 0.f;
    }
    template <bool EDGE>
    __device__ __forceinline__ void fetch(int64_t k0, int slot)
    {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            T e[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int64_t k = k0 + ch * 8 + j;
                const T v = g.p[min(k, K - 1) * g.s_k + min(row + i * kRowStep, last) * g.s_row];
                e[j] = k < K ? v : (T)0;
            }
            __builtin_memcpy(&raw[slot][i][0], e, sizeof(e));
        }
    }
    template <bool EDGE, bool TIMES>
    __device__ __forceinline__ void park(char *lds, int64_t, int slot)
    {
#pragma unroll
        for (int i = 0; i < PER; ++i) park_chunk<T, ROWS, TIMES>(lds, stage_offset<BK>(row + i * kRowStep, ch), raw[slot][i], lost, times);
    }
};

template <typename T>
struct ConvArgs {
    const T *x;
    int H, W, C, S, sh, sw, ph, pw, P, Q;
    uint32_t mC, mS, mPQ, mQ;  // multipliers for div_by
};

// The implicit im2col matrix of a convolution over NHWC x: row = output pixel (n, p, q), k = (r, s, c) with c
// fastest.  WHOLE: C is a multiple of 8, so a chunk lies inside one filter tap; else element loads.
template <typename T, int ROWS, int THREADS, int D, bool WHOLE>
struct ConvRows {
    using S = Split<T>;
    using Shallow = ConvRows<T, ROWS, THREADS, 1, WHOLE>;  // one register set
    static constexpr bool kElements = !WHOLE;  // loads element by element
    static constexpr int kDepth = D;
    static constexpr int BK = S::kBK, CH = BK / 8, ITEMS = ROWS * CH, PER = ITEMS / THREADS, V = 8 / S::kVec;
    static constexpr int kRowStep = THREADS / CH, kBlock = 1;
    static_assert(ITEMS % THREADS == 0 && kRowStep >= 16 && PER <= 4, "items divide among the threads, one chunk column per thread");
    using Args = ConvArgs<T>;
    Args g;
    int K, ch, o0;
    int64_t off[PER];  // element offset of the pixel under tap (0, 0), channel 0 (may lie outside x)
    int ih0[PER], iw0[PER];
    uint4_t raw[D][PER][WHOLE ? V : 2];  // the chunk, or its 8 elements one per word
    uint32_t ok[D];
    Lost lost;
    float times;
    int64_t first, pixels;

    __device__ __forceinline__ void pixel(int m, int &h0, int &w0, int64_t &o) const
    {
        const int n = div_by(m, g.P * g.Q, g.mPQ), pq = m - n * (g.P * g.Q);
        const int p = div_by(pq, g.Q, g.mQ), q = pq - p * g.Q;
        h0 = p * g.sh - g.ph;
        w0 = q * g.sw - g.pw;
        o = (((int64_t)n * g.H + h0) * g.W + w0) * g.C;
    }
    __device__ __forceinline__ float at(const Args &, int row, int64_t k) const
    {
        const bool real = first + row < pixels && k < K;
        int h0, w0, r, s, c;
        int64_t o;
        pixel((int)min(first + row, pixels - 1), h0, w0, o);
        tap((int)min(k, (int64_t)K - 1), r, s, c);
        const bool in = real && (unsigned)(h0 + r) < (unsigned)g.H && (unsigned)(w0 + s) < (unsigned)g.W;
        const float v = to_f32(g.x[in ? o + (int64_t)(r * g.W + s) * g.C + c : 0]);
        return in ? v : 0.f;
    }
    __device__ __forceinline__ void init(const Args &a, int64_t, int64_t r0, int64_t rows, int64_t K_, int tid)
    {
        g = a;
        K = (int)K_;
        first = r0;
        pixels = rows;
        ch = tid % CH;
        const int row = lds_row<BK>(tid / CH);
        o0 = stage_offset<BK>(row, ch);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            pixel((int)min(r0 + row + i * kRowStep, rows - 1), ih0[i], iw0[i], off[i]);
        }
    }
    __device__ __forceinline__ bool whole() const { return true; }
    __device__ __forceinline__ void tap(int k, int &r, int &s, int &c) const
    {
        const int t = div_by(k, g.C, g.mC);
        c = k - t * g.C;
        r = div_by(t, g.S, g.mS);
        s = t - r * g.S;
    }
    __device__ __forceinline__ bool inside(int i, int r, int s) const
    {
        return (unsigned)(ih0[i] + r) < (unsigned)g.H && (unsigned)(iw0[i] + s) < (unsigned)g.W;
    }
    template <bool EDGE>
    __device__ __forceinline__ void fetch(int64_t k0, int slot)
    {
        const int k = (int)k0 + ch * 8;
        uint32_t good = 0;
        if constexpr (WHOLE) {
            int r, s, c;
            tap(EDGE ? min(k, K - 8) : k, r, s, c);
            const int64_t d = (int64_t)(r * g.W + s) * g.C + c;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const bool in = (!EDGE || k < K) && inside(i, r, s);
                good |= in ? 1u << i : 0u;
                const T *p = g.x + (in ? off[i] + d : 0);
#pragma unroll
                for (int v = 0; v < V; ++v) raw[slot][i][v] = load_chunk<true>(p + v * S::kVec);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                int r, s, c;
                tap(EDGE ? min(k + j, K - 1) : k + j, r, s, c);
                const int64_t d = (int64_t)(r * g.W + s) * g.C + c;
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    const bool in = (!EDGE || k + j < K) && inside(i, r, s);
                    good |= in ? 1u << (8 * i + j) : 0u;
                    const T v = g.x[in ? off[i] + d : 0];
                    uint32_t w = 0;
                    __builtin_memcpy(&w, &v, sizeof(T));
                    raw[slot][i][j >> 2][j & 3] = w;
                }
            }
        }
        ok[slot] = good;
    }
    template <bool EDGE, bool TIMES>
    __device__ __forceinline__ void park(char *lds, int64_t, int slot)
    {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            uint4_t v[V];
            if constexpr (WHOLE) {
                const bool in = (ok[slot] >> i) & 1;
#pragma unroll
                for (int q = 0; q < V; ++q) v[q] = in ? raw[slot][i][q] : uint4_t{0u, 0u, 0u, 0u};
            } else {
                uint32_t w[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) w[j] = (ok[slot] >> (8 * i + j)) & 1 ? raw[slot][i][j >> 2][j & 3] : 0u;
                if constexpr (sizeof(T) == 2) {
#pragma unroll
                    for (int d = 0; d < 4; ++d) v[0][d] = w[2 * d] | (w[2 * d + 1] << 16);
                } else {
#pragma unroll
                    for (int d = 0; d < 8; ++d) v[d >> 2][d & 3] = w[d];
                }
            }
            park_chunk<T, ROWS, TIMES>(lds, stage_step<BK>(o0, i * kRowStep), v, lost, times);
        }
    }
};

// Workgroup id -> output tile: each XCD (ids are dealt round-robin to the 8 of them) gets a contiguous run of
// tiles, and runs walk the grid in column-major bands of 4 tile-rows (a compact patch shares operand panels).
__device__ __forceinline__ unsigned xcd_run(unsigned bid, unsigned total)
{
    const unsigned q = total / 8, rem = total % 8, xcd = bid % 8;
    return xcd * q + min(xcd, rem) + bid / 8;
}
__device__ __forceinline__ void band_tile(unsigned id, int tiles_m, int tiles_n, int &tm, int &tn)
{
    constexpr unsigned kBand = 4;
    const unsigned band = id / (kBand * (unsigned)tiles_n);
    const unsigned in_band = min(kBand, (unsigned)tiles_m - band * kBand);
    const unsigned within = id - band * kBand * (unsigned)tiles_n;
    tm = (int)(band * kBand + within % in_band);
    tn = (int)(within / in_band);
}

template <typename T, int TM, int TN, int WM, int WN, int KG>
struct StagedShape {
    using S = Split<T>;
    static constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN, kThreads = 64 * WM * WN;  // threads of one group
    static constexpr int kStageA = S::kPlanes * BM * 2 * S::kBK, kStageB = S::kPlanes * BN * 2 * S::kBK;
    static constexpr int kStage = kStageA + kStageB;
    static constexpr int kRed = KG > 1 ? (KG - 1) * BM * BN * 4 : 0;
    static constexpr int kLds = 2 * kStage * KG > kRed ? 2 * kStage * KG : kRed;
    static_assert(kLds <= 160 * 1024, "LDS of one CU");
    // as many workgroups of 4 waves as the LDS holds, three at most (registers for the loads in flight)
    static constexpr int kWavesPerSimd = kThreads * KG > 256 ? kThreads * KG / 256 : 160 * 1024 / kLds < 3 ? 160 * 1024 / kLds : 3;
};

template <typename ASrc, typename BSrc, typename T, typename CT, int TM, int TN, int WM, int WN, int KG, int D>
__global__ __launch_bounds__(64 * WM * WN * KG, (StagedShape<T, TM, TN, WM, WN, KG>::kWavesPerSimd)) void staged_kernel(typename ASrc::Args aa, typename BSrc::Args ba,
                                                                   CT *__restrict__ C, int64_t M, int64_t N, int64_t K,
                                                                   int64_t ldc, int64_t strideC, float alpha, int tiles_m,
                                                                   int tiles_n)
{
    using Shape = StagedShape<T, TM, TN, WM, WN, KG>;
    constexpr int NP = Split<T>::kPlanes, BK = Split<T>::kBK, BM = Shape::BM, BN = Shape::BN, NW = WM * WN;
    constexpr int U = D > 2 ? D : 2;  // rounds per pass of the loop: LDS stages and register sets are constants in it
    static_assert((D & (D - 1)) == 0 && (TM & (TM - 1)) == 0 && (TN & (TN - 1)) == 0, "powers of two");
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = KG > 1 ? wave_all / NW : 0, wave = KG > 1 ? wave_all % NW : wave_all;
    const int wm = wave / WN, wn = wave % WN;
    int tm, tn;
    band_tile(xcd_run(blockIdx.x, (unsigned)tiles_m * (unsigned)tiles_n), tiles_m, tiles_n, tm, tn);
    // A ragged last tile starts a few rows early if that lets it end on a whole block of its source.  The rows it shares
    // with its neighbour are the neighbour's to store: the two need not agree on them (one may have met a value that the
    // split does not hold), and an element has one writer.
    auto origin = [](int64_t r0, int64_t rows, int64_t edge, int block) {
        const int64_t over = rows - r0 < edge ? (rows - r0) % block : 0;
        return over != 0 && r0 > 0 ? r0 - (block - over) : r0;
    };
    const int64_t m0 = origin((int64_t)tm * BM, M, BM, ASrc::kBlock), n0 = origin((int64_t)tn * BN, N, BN, BSrc::kBlock);

    ASrc a_src;
    BSrc b_src;
    a_src.init(aa, blockIdx.y, m0, M, K, tid - group * Shape::kThreads);
    b_src.init(ba, blockIdx.y, n0, N, K, tid - group * Shape::kThreads);
    char *const mine = smem + group * 2 * Shape::kStage;
    const bool few_k = NP > 1 && K < 8;  // (no rounds: computed with the fp32 instruction)
    const int64_t nsteps = (K + BK - 1) / BK, rounds = few_k ? 0 : (nsteps + KG - 1) / KG;

    // Fragment addresses: tile rows 32 R + l, chunk 2 ks + lane / 32 sit at 32 R rows past the address of
    // rows l, chunk 2 (ks ^ R) + lane / 32: one register per k-substep and an immediate per tile.
    constexpr int KS = BK / 16;
    int fa[KS], fb[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        fa[ks] = wm * TM * 32 * 2 * BK + stage_offset<BK>(lane & 31, 2 * (ks ^ (wm * TM & (KS - 1))) + (lane >> 5));
        fb[ks] = Shape::kStageA + wn * TN * 32 * 2 * BK +
                 stage_offset<BK>(lane & 31, 2 * (ks ^ (wn * TN & (KS - 1))) + (lane >> 5));
    }
    WaveTile<TM, TN> t;
    t.clear();
    // One round's MFMAs from stage `buf`.  The fragments of a k-substep are read one substep ahead; hook(ks) is
    // issued behind those reads and before the substep's MFMAs (LDS accesses stay in program order, so a hook's
    // LDS writes must not stand in front of the reads that the next MFMAs wait for).
    auto multiply = [&](int buf, auto &&hook) {
        const char *stage = mine + buf * Shape::kStage;
        bf16x8_t a[2][NP][TM], b[2][NP][TN];
        auto read = [&](auto ks) {
#pragma unroll
            for (int p = 0; p < NP; ++p) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    a[ks & 1][p][i] =
                        *reinterpret_cast<const bf16x8_t *>(stage + fa[ks ^ (i & (KS - 1))] + (p * BM + i * 32) * (2 * BK));
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    b[ks & 1][p][j] =
                        *reinterpret_cast<const bf16x8_t *>(stage + fb[ks ^ (j & (KS - 1))] + (p * BN + j * 32) * (2 * BK));
            }
        };
        read(std::integral_constant<int, 0>{});
        unrolled<KS>([&](auto ks) {
            if constexpr (ks + 1 < KS) read(std::integral_constant<int, ks + 1>{});
            hook(ks);
            constexpr int c = ks & 1;
            if constexpr (NP == 1) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        t.acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[c][0][i], b[c][0][j], t.acc[i][j], 0, 0, 0);
            } else {
                constexpr int kPa[6] = {1, 0, 2, 0, 1, 0}, kPb[6] = {1, 2, 0, 1, 0, 0};  // the small products first
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int q = 0; q < 6; ++q)
                            t.acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[c][kPa[q]][i], b[c][kPb[q]][j], t.acc[i][j], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);  // (keeps a hook's global loads in its substep: the compiler sinks them to the end of the round)
        });
    };

    // Round `it`: the group's step it * KG + group is multiplied from stage it % 2, the next one goes from
    // register set (it + 1) % D to the other stage, and that set is refilled with step it + 1 + D.  Rounds are
    // straight-line code with no conditions around their loads (one that is issued on one of two paths makes
    // the compiler wait for all of them).
    // EDGE = false rounds: all that have only whole steps to fetch and park; if the rounds divide K, every one (what
    // they fetch past the end is the last step once more, never multiplied).
    const bool clean = a_src.whole() && b_src.whole(), even = K % (BK * KG) == 0;
    const int64_t fast_rounds = !clean ? 0 : even ? rounds : K / BK / KG - D - 1;
    auto step_k = [&](int64_t it) { return (it * KG + group) * BK; };
    // With one register set the start and the EDGE rounds skip fetches of steps that do not exist.  (Behind such a test all
    // loads are waited for, so it stands behind both parks.)
    constexpr bool kSkip = D == 1 && !ASrc::kElements && !BSrc::kElements;
    auto round = [&](auto &sa, auto &sb, auto u, auto edge, auto times, int64_t it) {
        constexpr int kD = std::remove_reference_t<decltype(sa)>::kDepth, slot = (u + 1) % kD, buf = u & 1;
        constexpr bool kEdge = decltype(edge)::value, kTimes = decltype(times)::value;
        char *la = mine + (buf ^ 1) * Shape::kStage, *lb = la + Shape::kStageA;
        const int64_t kp = step_k(it + 1), kn = kEdge ? step_k(it + 1 + kD) : min(step_k(it + 1 + kD), K - BK);
        constexpr bool kTest = kSkip && kEdge;
        multiply(buf, [&](auto ks) {
            if constexpr (ks == 0) {
                sa.template park<kEdge, kTimes>(la, kp, slot);
                if constexpr (!kTest) sa.template fetch<kEdge>(kn, slot);
            } else if constexpr (ks == 1) {
                sb.template park<kEdge, kTimes>(lb, kp, slot);
                if constexpr (!kTest) {
                    sb.template fetch<kEdge>(kn, slot);
                } else if (it + 1 + kD < rounds) {
                    sa.template fetch<kEdge>(kn, slot);
                    sb.template fetch<kEdge>(kn, slot);
                }
            }
        });
        __syncthreads();
    };
    auto start = [&](auto &sa, auto &sb, auto times, int64_t it) {
        constexpr int kD = std::remove_reference_t<decltype(sa)>::kDepth;
        constexpr bool kTimes = decltype(times)::value;
        unrolled<kD>([&](auto d) {
            sa.template fetch<true>(step_k(it + d), d);
            sb.template fetch<true>(step_k(it + d), d);
        });
        sa.template park<true, kTimes>(mine, step_k(it), 0);
        if constexpr (!kSkip) sa.template fetch<true>(step_k(it + kD), 0);
        sb.template park<true, kTimes>(mine + Shape::kStageA, step_k(it), 0);
        if (!kSkip || rounds > 1) {
            if constexpr (kSkip) sa.template fetch<true>(step_k(it + kD), 0);
            sb.template fetch<true>(step_k(it + kD), 0);
        }
        __syncthreads();
    };
    auto edge_rounds = [&](auto &sa, auto &sb, auto times, int64_t it) {
        constexpr int kD = std::remove_reference_t<decltype(sa)>::kDepth;
        while (it < rounds) {
            bool more = true;
            unrolled<(kD > 2 ? kD : 2)>([&](auto u) {
                if (more) {
                    round(sa, sb, u, std::true_type{}, times, it);
                    more = ++it < rounds;
                }
            });
        }
    };
    if (D > 1 || !few_k) start(a_src, b_src, std::false_type{}, 0);  // (few k come to kernels with one register set)
    int64_t it = 0;
    for (; it + U <= fast_rounds; it += U)
        unrolled<U>([&](auto u) { round(a_src, b_src, u, std::false_type{}, std::false_type{}, it + u); });
    edge_rounds(a_src, b_src, std::false_type{}, it);
    bool direct = false;  // the fp32 matrix instruction, operands straight from memory
    if constexpr (NP > 1) {
        auto not_finite = [&]() {
            float z = 0.f;  // (infinities and NaN make it NaN)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) z = __builtin_fmaf(t.acc[i][j][e], 0.f, z);
            return z != 0.f;
        };
        const bool lost_a = a_src.lost.any(), lost_b = b_src.lost.any(), no_sum = few_k || not_finite();
        if (__syncthreads_or(lost_a || lost_b || no_sum)) {
            const float times_a = __syncthreads_or(lost_a) ? 0x1p24f : 1.f, times_b = __syncthreads_or(lost_b) ? 0x1p24f : 1.f;
            direct = __syncthreads_or(no_sum) != 0;
            // (everything anew, from values that the compiler takes for others: what it would keep costs the loop above registers)
            int tid2 = tid;
            int64_t K2 = K, first = 0;
            asm volatile("" : "+v"(tid2), "+s"(K2), "+s"(first));
            typename ASrc::Shallow a2;
            typename BSrc::Shallow b2;
            a2.init(aa, blockIdx.y, m0, M, K2, tid2 - group * Shape::kThreads);
            b2.init(ba, blockIdx.y, n0, N, K2, tid2 - group * Shape::kThreads);
            // A value loses less than 2^-133, so a sum less than 2^-133 K max |other operand|: nothing that shows if every sum
            // is 2^28 times that.  (Probabilities times values: those that underflow stand beside others.)
            bool again = !direct;
            if (KG == 1 && again) {
                auto largest = [&](auto &src) {
                    float m = 0.f;
                    for (int64_t k = first; k < K2; k += BK) {
                        src.template fetch<true>(k, 0);
                        const uint4_t(&w)[sizeof(src.raw[0]) / 16] = reinterpret_cast<const uint4_t(&)[sizeof(src.raw[0]) / 16]>(src.raw[0]);
#pragma unroll
                        for (unsigned i = 0; i < sizeof(src.raw[0]) / 16; ++i)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const uint32_t bits = w[i][e];
                                m = __builtin_fmaxf(m, __builtin_fabsf(__builtin_bit_cast(float, bits)));
                            }
                    }
                    return m;
                };
                float big = 0.f;
                if (times_a > 1.f) big = largest(b2);
                if (times_b > 1.f) big = __builtin_fmaxf(big, largest(a2));
                big = wave_allreduce(big, OpMax{});
                float *red = reinterpret_cast<float *>(smem);  // (no stage is read any more)
                if ((tid2 & 63) == 0) red[wave_all] = big;
                __syncthreads();
#pragma unroll
                for (int w = 0; w < NW; ++w) big = __builtin_fmaxf(big, red[w]);
                const float least = 0x1p-104f * (float)K * big;  // (2^29 times: both operands may have lost)
                bool small = false;
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int e = 0; e < 16; ++e) small |= !(__builtin_fabsf(t.acc[i][j][e]) >= least);
                again = __syncthreads_or(small) != 0;
            }
            if (again) {
                a2.times = times_a;
                b2.times = times_b;
                t.clear();
                start(a2, b2, std::true_type{}, first);
                edge_rounds(a2, b2, std::true_type{}, first);
                direct = __syncthreads_or(not_finite()) != 0;
                const float back = (times_a > 1.f ? 0x1p-24f : 1.f) * (times_b > 1.f ? 0x1p-24f : 1.f);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int e = 0; e < 16; ++e) t.acc[i][j][e] *= back;
            }
            if (direct && group == 0) {
                const int l = tid2 & 63;
                t.clear();
                for (int64_t k = l >> 5; k < K + (l >> 5); k += 2) {  // (the same count in both halves of the wave)
                    float a[TM], b[TN];
#pragma unroll
                    for (int i = 0; i < TM; ++i) a[i] = a2.at(aa, (wm * TM + i) * 32 + (l & 31), k);
#pragma unroll
                    for (int j = 0; j < TN; ++j) b[j] = b2.at(ba, (wn * TN + j) * 32 + (l & 31), k);
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j) t.acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], t.acc[i][j], 0, 0, 0);
                }
            }
        }
    }
    if (direct) {
        if (group > 0) return;
    } else if constexpr (KG > 1) {
        // the groups' sums, added in group order
        float *red = reinterpret_cast<float *>(smem);
        if (group > 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        red[((((group - 1) * NW + wave) * TM * TN + i * TN + j) * 16 + e) * 64 + lane] = t.acc[i][j][e];
        }
        __syncthreads();
        if (group > 0) return;
#pragma unroll
        for (int h = 0; h < KG - 1; ++h)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        t.acc[i][j][e] += red[(((h * NW + wave) * TM * TN + i * TN + j) * 16 + e) * 64 + lane];
    }
    CT *Ct = C + (int64_t)blockIdx.y * strideC + m0 * ldc + n0;
    constexpr bool kEarly = ASrc::kBlock > 1 || BSrc::kBlock > 1;  // (tiles that can start early)
    store_tile<TM, TN, CT, kEarly>(t, Ct, ldc, (int)min((int64_t)BM, M - m0), (int)min((int64_t)BN, N - n0), wm * 32 * TM, wn * 32 * TN,
                           alpha, lane, (int)((int64_t)tm * BM - m0), (int)((int64_t)tn * BN - n0));
}

struct GemmArgs {
    const void *A, *B;
    void *C;
    int64_t M, N, K, lda, ldb, ldc, batch, strideA, strideB, strideC;
    int la, lb;
    float alpha;
    hipStream_t st;
};

// A convolution as launch_staged_conv takes it: NHWC x, KRSC w, NPQK y.  (ph may be negative: rows p0 .. of an image are a
// convolution with ph - p0 sh.)
struct StagedConv {
    const void *x, *w;
    void *y;
    int N, H, W, C, K, R, S, sh, sw, ph, pw, P, Q;
    hipStream_t st;
};

// Any stride, padding, channel count and type (staged_conv.hip).
perf_status launch_staged_conv(const StagedConv &c, int xw_dt, int y_dt);

// The kernels whose waves divide the reduction (waves_conv.hip): false if they do not suit the call.  direct: the
// convolution's own main loop takes it as well.
bool launch_waves_conv(const StagedConv &c, int xw_dt, int y_dt, bool direct, perf_status *status);

// Any layout, type (ab: bf16 or fp32 operands), size and alignment (staged_gemm.hip).
perf_status launch_staged_gemm(const GemmArgs &g, int ab_dt, int c_dt);

// The kernels whose waves divide K (waves_gemm.hip): false if they do not suit the call.  direct: the direct kernels of
// gemm.hip take it as well.
bool launch_waves_gemm(const GemmArgs &g, int ab_dt, int c_dt, bool direct, perf_status *status);

}  // namespace perf
