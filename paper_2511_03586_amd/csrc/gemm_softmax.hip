// Attention-score GEMM with the row softmax as its epilogue, for gfx950:
//     P_b = softmax_rows(alpha * A_b * B_b^T)
// (the "bmm" and "softmax" rows of the operator table, Section 4.3 of the paper, joined the
// way the paper's fusion moves join producer and consumer scopes, Sections 2.2 and 3.1: the
// score matrix never goes to memory, so the traffic is the operands plus one write of P).
//
//  * gemm_softmax_kernel: bf16 operands, both K-contiguous, K = 64, N = 128, 256 or 512 (K = 128: N = 128), fp32 P.  A
//    workgroup of 8 waves takes strips of 128 rows x all N columns of one matrix; each wave 16 rows x N
//    as up to 32 accumulators of 16x16 (128 registers), computed with B as the MFMA's row
//    operand, so that a lane holds 4 consecutive columns per accumulator and all of a
//    lane's values belong to ONE row: the row reductions are in-lane plus two lane
//    exchanges.  The operand strips and all of B go to LDS (global->LDS loads, the swizzled 128-byte rows
//    of mfma_tile.h): B once per workgroup, which then walks over several row strips of the
//    matrix with the next strip's rows in flight.
//  * gemm_softmax_wide_kernel: bf16 operands, any K that is a multiple of 8 up to 512, N <= 1024, P of any
//    alignment: strips of 32 rows, B streamed through the LDS.
//  * any other legal case: perf_gemm into P followed by perf_softmax in place.
#include <atomic>
#include "mfma_tile.h"
#include "row_io.h"
#include "softmax_math.h"
#include "host_utils.h"

namespace perf {

// T16N: 16-column accumulators per wave (N = 16 * T16N, a multiple of 128).
// A workgroup takes `group` consecutive row strips of one matrix: B goes to LDS once per
// workgroup, and a wave's 16 rows of the next strip are fetched (into the other of two
// buffers; the rows are the wave's own, so no barrier is involved) while it works on the
// present one, so its stores follow each other without a load latency in between.
// One workgroup per CU: the probabilities leave through a private 8 KiB LDS region per wave, 128 columns at a time, so that a store instruction writes 2 rows x
// 512 contiguous bytes instead of 8 rows x 128.  A write-only probe of this output (a wave writing its 16
// rows of 2 KiB per strip) moves 5.6 TB/s in the first shape and 6.3 in the second (6.4 with 1 KiB per row,
// for which the LDS has no room): the shape of the store instruction, not the exponentials, held the
// kernel at 0.68 of the HBM peak.
constexpr int kFusedWaves = 8;
template <int T16N>
__global__ __launch_bounds__(64 * kFusedWaves, 1) void gemm_softmax_kernel(const uint16_t *__restrict__ A,
                                                              const uint16_t *__restrict__ B, float *__restrict__ P,
                                                              int M, int N, int K, int64_t lda, int64_t ldb,
                                                              int64_t ldp, int64_t strideA, int64_t strideB,
                                                              int64_t strideP, float sign, float c, int strips,
                                                              int group, int xcd_remap)
{
    constexpr int NW = kFusedWaves, BM = 16 * NW, BN = 16 * T16N;
    static_assert(T16N % 8 == 0, "the staged write-out takes whole chunks of 128 columns");
    constexpr int LB = (BN + 8 * NW - 1) / (8 * NW);     // wave loads per K-step of 64 for B (the last one may be partly unused)
    constexpr int kRowsB = LB * 8 * NW;
    constexpr int kStepB = kRowsB * kRowBytes64, kStepA = BM * kRowBytes64;
    extern __shared__ __attribute__((aligned(1024))) char smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: LDS addresses stay scalar
    // Workgroup id -> (strip group, matrix).  Ids are dealt round-robin to the 8 XCDs, each with
    // a private L2; with the remap all groups of one matrix run on one XCD, so B is fetched
    // over the fabric once per matrix.
    const int groups = (strips + group - 1) / group;
    int gi, bz;
    if (xcd_remap) {
        const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
        gi = j % groups;
        bz = (j / groups) * 8 + xcd;
    } else {
        gi = blockIdx.x % groups;
        bz = blockIdx.x / groups;
    }
    const int s0 = gi * group, s1 = min(strips, s0 + group);
    const int ksteps = K / 64;
    const uint16_t *Ab = A + (int64_t)bz * strideA;
    const uint16_t *Bb = B + (int64_t)bz * strideB;
    float *Pb = P + (int64_t)bz * strideP;
    char *const smem_a = smem + ksteps * kStepB;  // two buffers of ksteps x BM rows
    char *const stage = smem_a + 2 * ksteps * kStepA + wave * (16 * 512);  // this wave's 16 rows x 128 columns

    // this wave's 16 rows of strip s -> buffer s & 1 (nothing if the rows lie past M)
    auto issue_a = [&](int s) {
        const int row0 = s * BM + wave * 16;
        if (row0 >= M) return;
        RowMajorSrc64<2, 1> src(Ab + (int64_t)row0 * lda, min(16, M - row0), lda, ksteps, 0, lane);
        char *buf = smem_a + (s & 1) * ksteps * kStepA + wave * 16 * kRowBytes64;
        for (int ks = 0; ks < ksteps; ++ks) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint32_t vo = src.voff[i], so = src.soff;
                issue_load_to(src.rsrc, vo, so, buf + ks * kStepA + i * 8 * kRowBytes64);
            }
            src.advance();
        }
    };

    {
        RowMajorSrc64<LB, NW> src_b(Bb, min(kRowsB, N), ldb, ksteps, wave, lane);
        for (int ks = 0; ks < ksteps; ++ks) {
#pragma unroll
            for (int i = 0; i < LB; ++i) {
                const uint32_t vo = src_b.voff[i], so = src_b.soff;
                issue_load_to(src_b.rsrc, vo, so, smem + ks * kStepB + (i * NW + wave) * 8 * kRowBytes64);
            }
            src_b.advance();
        }
    }
    issue_a(s0);
    wait_vmem<0>();
    wg_barrier();  // B is complete (and each wave's own rows of the first strip)

    for (int s = s0; s < s1; ++s) {
        if (s + 1 < s1) issue_a(s + 1);
        const int m0 = s * BM;
        if (m0 + wave * 16 >= M) continue;  // (no barrier inside the loop)
        const char *abuf = smem_a + (s & 1) * ksteps * kStepA;
        // acc[j] element e: row m0 + 16*wave + lane%16, column 16 j + 4 (lane/16) + e
        WaveTile16<1, T16N> t;
        t.clear();
        for (int ks = 0; ks < ksteps; ++ks) {
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const int chunk = 4 * half + (lane >> 4);
                const bf16x8_t a =
                    *reinterpret_cast<const bf16x8_t *>(abuf + ks * kStepA + frag_offset64(wave * 16 + (lane & 15), chunk));
#pragma unroll
                for (int j = 0; j < T16N; ++j) {
                    const bf16x8_t b = *reinterpret_cast<const bf16x8_t *>(smem + ks * kStepB +
                                                                            frag_offset64(j * 16 + (lane & 15), chunk));
                    t.acc[0][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a, t.acc[0][j], 0, 0, 0);
                }
            }
        }
        // the reads of this strip's rows are back before the buffer is refilled two strips on
        // (the compiler waits for them in front of the MFMAs that use them)

        // Row softmax.  All of a lane's values belong to row lane%16; lanes l, l^16, l^32, l^48
        // share it.  exp(|alpha| * (v - m)) is evaluated as exp2 of a plain product: its relative
        // error is ~2^-24 times the exponent, i.e. below 4e-6 for every result above 2^-100, and
        // smaller results are below the floor under which only the absolute error is specified.
        float m = -FLT_MAX;
#pragma unroll
        for (int j = 0; j < T16N; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float v = t.acc[0][j][e] * sign;
                t.acc[0][j][e] = v;
                m = __builtin_fmaxf(m, v);
            }
        {
            float a, b;
            swap16(m, a, b);
            m = __builtin_fmaxf(a, b);
            swap32(m, a, b);
            m = __builtin_fmaxf(a, b);
        }
        float z = 0.f;
#pragma unroll
        for (int j = 0; j < T16N; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float p = __builtin_amdgcn_exp2f((t.acc[0][j][e] - m) * c);
                t.acc[0][j][e] = p;
                z += p;
            }
        {
            float a, b;
            swap16(z, a, b);
            z = a + b;
            swap32(z, a, b);
            z = a + b;
        }
        const float scale = 1.0f / z;
        // The next strip's rows must have landed before they are read: waiting here, in front of this strip's
        // stores, leaves those in flight across the next strip's MFMAs.  (Letting two strips of stores stay in
        // flight, by waiting for a count at the top of the loop instead, measured no faster.)
        wait_vmem<0>();
        {
            // 128 columns at a time: lane (row r = lane % 16, q = lane / 16) writes its 16-byte pieces 4 jj + q of
            // the chunk to row r of the staging; a row is 32 pieces, piece s at position s ^ r (then both the
            // writes, 16 rows per quarter-wave, and the reads, 16 consecutive pieces of a row, are conflict
            // free at a pitch of 512 bytes); then 8 instructions read and store 2 rows x 512 bytes each.
            const int r = lane & 15, q = lane >> 4, piece = lane & 31, half = lane >> 5;
            const int64_t row_base = (int64_t)(m0 + wave * 16);
#pragma unroll
            for (int ch = 0; ch < T16N / 8; ++ch) {
#pragma unroll
                for (int jj = 0; jj < 8; ++jj) {
                    const float4_t v = t.acc[0][8 * ch + jj] * scale;
                    *reinterpret_cast<float4_t *>(stage + r * 512 + (((4 * jj + q) ^ r) << 4)) = v;
                }
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): own writes are in LDS (the region is this wave's alone)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int R = 2 * i + half;
                    const float4_t v = *reinterpret_cast<const float4_t *>(stage + R * 512 + ((piece ^ R) << 4));
                    if (row_base + R < M)
                        __builtin_nontemporal_store(v, reinterpret_cast<float4_t *>(Pb + (row_base + R) * ldp + ch * 128 + piece * 4));
                }
            }
        }
    }
}

// Longer and ragged rows: N <= 1024, K any multiple of 8, P of any alignment.  A workgroup of NW waves owns 32 rows x all N
// columns; wave w the NT tiles of 32 columns from 32 NT w on, as 32x32 accumulators with B as the MFMA's row operand, so
// that a lane's values belong to ONE row: row maxima and sums are in-lane plus one lane exchange, and one LDS exchange
// between the waves.  Both operands come 32 K at a time (chunks past K read as zeros), B once per strip from the L2:
//   * OWN: a wave loads the rows of B that it multiplies itself, reads a step's operands into registers and refills the
//     stage in front of its matrix instructions, without a barrier (80 x (512x384x64) 17.8 against 19.6 on shared stages).  It takes
//     24 registers and more that the shared stages do not.  <4, float, 8, true> has one too few for its eight addresses of B and
//     reloads one of them in each step, which waits for the step's other loads.
//   * else through the LDS that all waves fill, two stages for NT <= 2 (400 x (200x100x80) 13.2 us against 15.7 with OWN), one above.
// At most 80 KiB of LDS, so that two workgroups or more share a CU and one's loads and exponentials overlap the other's
// stores; eight waves where there are registers for them (the fp32 instructions of an exponential issue twice as fast from two
// waves of a SIMD as from one): 96 x (600x800x80) 60 us against 63, 60 x (100x450x128) 9.6 against 11.3.
// Write-out: 16 or 32 rows at a time through the LDS, so that a wave stores whole rows, 1 KiB of consecutive bytes per instruction,
// past the caches.  With 256 bytes of four rows per instruction the lines that two of them share had to be put together in
// the L2: 96 x (600x777x80) 82 us against 65 now, 80 x (512x384x64), whose rows are whole lines, 24.5 against 17.8,
// 64 x (1000x1024x128) 106 against 74, 400 x (200x100x80) 18.7 against 13.2.  (Two store instructions that differ in the cache
// policy alone, on the two sides of a test, are merged by the compiler into one of the plain kind.)  Up to 16 rows of a strip
// are dealt to the waves one by one: 128 x (6x192x32) 4.56 us with all of them stored by the first wave, 4.32.
//   * FEW: a P that the caches hold leaves from the registers (plain stores, 16 bytes of a row per lane) without the LDS's latency and
//     two barriers: 360 x (32x13x80) 4.22 -> 3.96 us, 155 x (22x56x16) 3.35 -> 3.14, bf16 P 43 x (48x35x128) 4.32 -> 3.94.
// The first shape's P is 28 us of writes at the copy rate, its exponentials about 15 us of vector work.
constexpr int wide_stages(int nt) { return nt <= 2 ? 2 : 1; }      // that all waves fill
constexpr int wide_rows_out(int nt) { return nt > 2 ? 16 : 32; }  // as the LDS of the operands holds them
template <int NT, typename PT, int NW, bool OWN, bool FEW>
__global__ __launch_bounds__(64 * NW, NW == 8 ? 4 : 2) void gemm_softmax_wide_kernel(const uint16_t *__restrict__ A, const uint16_t *__restrict__ B,
                                                                   PT *__restrict__ P, int M, int N, int K, int64_t lda,
                                                                   int64_t ldb, int64_t ldp, int64_t strideA, int64_t strideB,
                                                                   int64_t strideP, ExpConst ek, float t_min, int strips, int eights)
{
    constexpr int kStage = (OWN ? 32 * NT : 32 * NW * NT + 32) * kRowBytes, LB = 2 * NT, NST = wide_stages(NT);
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    __shared__ float red[2][NW][32];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (all strips of a matrix on one XCD, but for the last matrices of a batch that 8 does not divide: B comes over the fabric once)
    int si, bz;
    if ((int)blockIdx.x < eights * 8 * strips) {
        const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
        si = j % strips;
        bz = (j / strips) * 8 + xcd;
    } else {
        si = blockIdx.x % strips;
        bz = blockIdx.x / strips;
    }
    const int m0 = si * 32, ksteps = (K + 31) / 32, rows = min(32, M - m0);
    const uint16_t *Ab = A + (int64_t)bz * strideA + (int64_t)m0 * lda;
    const uint16_t *Bb = B + (int64_t)bz * strideB;
    const rsrc_t ra = make_rsrc(Ab, (uint32_t)(((int64_t)(rows - 1) * lda + K) * 2));
    const rsrc_t rb = make_rsrc(Bb, (uint32_t)(((int64_t)(N - 1) * ldb + K) * 2));

    const int lrow = lane >> 2, kb = load_chunk(lrow, lane) * 8;  // a load: 16 rows, lane l row l / 4, the chunk stored at position l % 4
    float16_t acc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;
    if constexpr (!OWN) {
        // load i of wave w: rows (NW i + w) * 16 .. + 15 of B
        uint32_t vb[LB];
#pragma unroll
        for (int i = 0; i < LB; ++i) vb[i] = (uint32_t)(min((i * NW + wave) * 16 + lrow, N - 1) * ldb * 2) + kb * 2;
        const uint32_t va = (uint32_t)(min((wave & 1) * 16 + lrow, rows - 1) * lda * 2) + kb * 2;
        auto issue = [&](int ks) {
            char *st = smem + (NST == 2 ? (ks & 1) * kStage : 0);
            const bool in = ks * 32 + kb < K;
            const uint32_t so = (uint32_t)ks * kRowBytes;
#pragma unroll
            for (int i = 0; i < LB; ++i) issue_load_to(rb, in ? vb[i] : kOutOfRange, so, st + (i * NW + wave) * 16 * kRowBytes);
            issue_load_to(ra, in ? va : kOutOfRange, so, st + (32 * NW * NT + (wave & 1) * 16) * kRowBytes);  // (waves 2 on: the same again)
        };
        issue(0);
        if (NST == 2 && ksteps > 1) issue(1);
        for (int ks = 0; ks < ksteps; ++ks) {
            if (NST == 2 && ks + 1 < ksteps) wait_vmem<LB + 1>();
            else wait_vmem<0>();
            wg_barrier();
            const char *st = smem + (NST == 2 ? (ks & 1) * kStage : 0);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int chunk = 2 * h + (lane >> 5);
                const bf16x8_t a = *reinterpret_cast<const bf16x8_t *>(st + frag_offset(32 * NW * NT + (lane & 31), chunk));
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const bf16x8_t b = *reinterpret_cast<const bf16x8_t *>(st + frag_offset((wave * NT + j) * 32 + (lane & 31), chunk));
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, acc[j], 0, 0, 0);
                }
            }
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave is done with the stage
            wg_barrier();
            if (ks + NST < ksteps) issue(ks + NST);
        }
    } else {
        // load i: rows 16 i .. + 15 of the wave's own columns; the rows of A come straight into the matrix instruction's layout
        char *const st = smem + wave * kStage;
        const int tiles = min(max((N - 32 * wave * NT + 31) / 32, 0), NT);  // those that have columns
        uint32_t vb[LB];
#pragma unroll
        for (int i = 0; i < LB; ++i) vb[i] = (uint32_t)(min(32 * wave * NT + 16 * i + lrow, N - 1) * ldb * 2) + kb * 2;
        const uint32_t va = (uint32_t)(min(lane & 31, rows - 1) * lda * 2) + (lane >> 5) * 16;
        bf16x8_t a[2], b[2][NT], next[2];
        auto issue = [&](int ks) {
            const bool in = ks * 32 + kb < K;
            const uint32_t so = (uint32_t)ks * kRowBytes;
#pragma unroll
            for (int i = 0; i < LB; ++i)
                if (i / 2 < tiles) issue_load_to(rb, in ? vb[i] : kOutOfRange, so, st + i * 16 * kRowBytes);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t from = ks * 32 + 16 * h + 8 * (lane >> 5) < K ? va + 32 * h : kOutOfRange;
                next[h] = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(ra, from, so, 0));
            }
        };
        issue(0);
        for (int ks = 0; ks < ksteps; ++ks) {
            wait_vmem<0>();
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                a[h] = next[h];
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    b[h][j] = *reinterpret_cast<const bf16x8_t *>(st + frag_offset(j * 32 + (lane & 31), 2 * h + (lane >> 5)));
            }
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave is done with the stage
            if (ks + 1 < ksteps) issue(ks + 1);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[h][j], a[h], acc[j], 0, 0, 0);
        }
    }

    // acc[j] element e: row m0 + lane % 32, column 32 (wave NT + j) + 8 (e / 4) + 4 (lane / 32) + e % 4
    const int row = lane & 31, half = lane >> 5, col0 = 32 * wave * NT;
    if (ek.sign < 0.f) {  // (uniform: the maximum of -v)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[j][e] = -acc[j][e];
    }
    auto column = [&](int j, int e) { return col0 + 32 * j + 8 * (e >> 2) + 4 * half + (e & 3); };
    const bool ragged = col0 + 32 * NT > N;  // (uniform) some of this wave's columns lie past N
    if (ragged) {
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[j][e] = column(j, e) < N ? acc[j][e] : -FLT_MAX;
    }
    float m = -FLT_MAX;
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) m = __builtin_fmaxf(m, acc[j][e]);
    float x, y;
    swap32(m, x, y);
    red[0][wave][row] = __builtin_fmaxf(x, y);  // (both halves write the same)
    __syncthreads();
    m = red[0][0][row];
#pragma unroll
    for (int w = 1; w < NW; ++w) m = __builtin_fmaxf(m, red[0][w][row]);
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] = exp_scaled_above(acc[j][e] - m, ek.c_hi, ek.c_lo, t_min);
    if (ragged) {  // (scale 0 would give masked columns weight 1)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[j][e] = column(j, e) < N ? acc[j][e] : 0.f;
    }
    float z = 0.f;
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) z += acc[j][e];
    swap32(z, x, y);
    red[1][wave][row] = x + y;
    __syncthreads();  // (behind it the operand stages are free)
    float part[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) part[w] = red[1][w][row];
#pragma unroll
    for (int d = 1; d < NW; d *= 2)
#pragma unroll
        for (int w = 0; w + d < NW; w += 2 * d) part[w] += part[w + d];
    const float sum = part[0];
    const float inv = 1.0f / sum;

    auto store = [&](PT *dst, float4_t v, int left) {  // `left` columns of the row from here on
        if (left >= 4) {
            if constexpr (sizeof(PT) == 4) {
                if constexpr (FEW) *reinterpret_cast<float4_at4 *>(dst) = v;
                else __builtin_nontemporal_store(v, reinterpret_cast<float4_at4 *>(dst));
            } else {
                const uint2_t o = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
                if constexpr (FEW) *reinterpret_cast<uint2_at2 *>(dst) = o;
                else __builtin_nontemporal_store(o, reinterpret_cast<uint2_at2 *>(dst));
            }
        } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (e < left) Elem<PT>::store1(dst + e, v[e]);
        }
    };
    PT *Pb = P + (int64_t)bz * strideP + (int64_t)m0 * ldp;
    if (FEW && rows > 16) {  // straight from the registers
        if (row < rows) {
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4_t v = {acc[j][4 * q] * inv, acc[j][4 * q + 1] * inv, acc[j][4 * q + 2] * inv, acc[j][4 * q + 3] * inv};
                    const int col = column(j, 4 * q);
                    store(Pb + (int64_t)row * ldp + col, v, N - col);
                }
        }
        return;
    }
    // Write-out, kOut rows at a time through the LDS of the operands.  kPieces pieces of 16 bytes per row, piece s at
    // position s ^ row.
    constexpr int kOut = wide_rows_out(NT), kPieces = 8 * NT * NW, kPitch = 16 * kPieces;
    constexpr int kRowsPer = kPieces < 64 ? 64 / kPieces : 1;  // rows per store instruction
#pragma unroll
    for (int pass = 0; pass < 32 / kOut; ++pass) {
        if (pass > 0) __syncthreads();  // the rows before have been read
        if (row / kOut == pass) {
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4_t v = {acc[j][4 * q] * inv, acc[j][4 * q + 1] * inv, acc[j][4 * q + 2] * inv, acc[j][4 * q + 3] * inv};
                    const int piece = 8 * (wave * NT + j) + 2 * q + half;
                    *reinterpret_cast<float4_t *>(smem + row % kOut * kPitch + ((piece ^ (row & 15)) << 4)) = v;
                }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kOut / NW / kRowsPer; ++i) {
            // (a wave's rows lie one after the other; few of them are dealt out)
            const int r = (rows > 16 ? wave * (kOut / NW) + i * kRowsPer : (i * NW + wave) * kRowsPer) + (kRowsPer > 1 ? lane / kPieces : 0);
            if (pass * kOut + r < rows) {
                PT *to = Pb + (int64_t)(pass * kOut + r) * ldp;
#pragma unroll
                for (int p0 = 0; p0 < kPieces; p0 += 64) {
                    const int piece = kRowsPer > 1 ? lane % kPieces : p0 + lane, left = N - 4 * piece;  // columns from here on
                    if (left > 0)
                        store(to + 4 * piece, *reinterpret_cast<const float4_t *>(smem + r * kPitch + ((piece ^ (r & 15)) << 4)), left);
                }
            }
        }
    }
}

template <int NT, typename PT, int NW = 4, bool OWN = false, bool FEW = false>
static perf_status launch_wide(const void *A, const void *B, void *P, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb,
                               int64_t ldp, int64_t batch, int64_t strideA, int64_t strideB, int64_t strideP, float alpha,
                               hipStream_t st)
{
    constexpr int kStages = OWN ? 32 * NW * NT * kRowBytes : wide_stages(NT) * (32 * NW * NT + 32) * kRowBytes, kOut = wide_rows_out(NT) * 128 * NT * NW;
    constexpr int kLds = kStages > kOut ? kStages : kOut;
    auto kern = gemm_softmax_wide_kernel<NT, PT, NW, OWN, FEW>;
    static std::atomic<bool> attr_done{false};  // (idempotent per-function setting)
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kLds) != hipSuccess)
            return PERF_ERR_LAUNCH;
        attr_done = true;
    }
    const ExpConst ek = make_exp_const(alpha);
    const float t_min = ek.c_hi > 0.f ? std::fmax(-200.0f / ek.c_hi, -FLT_MAX) : -FLT_MAX;
    const int64_t strips = (M + 31) / 32, per_launch = (max_blocks(64 * NW) / strips) / 8 * 8;
    if (per_launch < 8) return PERF_ERR_UNSUPPORTED;
    for (int64_t b0 = 0; b0 < batch; b0 += per_launch) {
        const int64_t nb = batch - b0 < per_launch ? batch - b0 : per_launch;
        hipLaunchKernelGGL(kern, dim3((unsigned)(strips * nb)), dim3(64 * NW), kLds, st, (const uint16_t *)A + b0 * strideA,
                           (const uint16_t *)B + b0 * strideB, (PT *)P + b0 * strideP, (int)M, (int)N, (int)K, lda, ldb, ldp,
                           strideA, strideB, strideP, ek, t_min, (int)strips, (int)(nb / 8));
    }
    return launch_status();
}

// gemm_softmax_kernel: 8 waves, 128-row strips, 160 KiB of LDS (B 64 KiB, two row buffers of 16 KiB, 64 KiB of staging).
template <int T16N>
static perf_status launch_fused_staged(const void *A, const void *B, void *P, int64_t M, int64_t N, int64_t K, int64_t lda,
                                       int64_t ldb, int64_t ldp, int64_t batch, int64_t strideA, int64_t strideB,
                                       int64_t strideP, float alpha, hipStream_t st)
{
    constexpr int NW = kFusedWaves;
    constexpr int kRowsB = (16 * T16N + 8 * NW - 1) / (8 * NW) * (8 * NW);
    const size_t lds = (size_t)(K / 64) * (2 * 16 * NW + kRowsB) * kRowBytes64 + (size_t)NW * 16 * 512;
    if (lds > 160 * 1024) return PERF_ERR_UNSUPPORTED;
    auto kern = gemm_softmax_kernel<T16N>;
    static std::atomic<bool> attr_done{false};  // (idempotent per-function setting)
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                160 * 1024) != hipSuccess)
            return PERF_ERR_LAUNCH;
        attr_done = true;
    }
    const float sign = alpha < 0.f ? -1.f : 1.f;
    const float c = (float)(std::fabs((double)alpha) * 1.4426950408889634074);  // |alpha| log2(e)
    const int64_t strips = (M + 16 * NW - 1) / (16 * NW);
    // strips per workgroup: as many as still leave two workgroups for every CU (one runs at a time)
    int64_t group = strips * batch / 512;
    group = group < 1 ? 1 : group > strips ? strips : group;
    const int64_t groups = (strips + group - 1) / group;
    const int64_t per_launch = (max_blocks(64 * NW) / groups) / 8 * 8;
    if (per_launch < 8) return PERF_ERR_UNSUPPORTED;
    for (int64_t b0 = 0; b0 < batch; b0 += per_launch) {
        const int64_t nb = batch - b0 < per_launch ? batch - b0 : per_launch;
        hipLaunchKernelGGL(kern, dim3((unsigned)(groups * nb)), dim3(64 * NW), lds, st, (const uint16_t *)A + b0 * strideA,
                           (const uint16_t *)B + b0 * strideB, (float *)P + b0 * strideP, (int)M, (int)N, (int)K, lda, ldb,
                           ldp, strideA, strideB, strideP, sign, c, (int)strips, (int)group, nb % 8 == 0 ? 1 : 0);
    }
    return launch_status();
}

}  // namespace perf

extern "C" perf_status perf_gemm_softmax(const void *A, const void *B, void *P, int64_t M, int64_t N, int64_t K,
                                         int64_t lda, int64_t ldb, int64_t ldp, int64_t batch, int64_t strideA,
                                         int64_t strideB, int64_t strideP, float alpha, perf_dtype ab_dt,
                                         perf_dtype p_dt, perf_stream stream)
{
    using namespace perf;
    if (!A || !B || !P) return PERF_ERR_NULL;
    if (!dtype_ok(ab_dt) || !dtype_ok(p_dt)) return PERF_ERR_DTYPE;
    if (M < 1 || N < 1 || K < 1 || batch < 1) return PERF_ERR_SHAPE;
    if (lda < K || ldb < K || ldp < N) return PERF_ERR_SHAPE;
    if (strideA < 0 || strideB < 0 || strideP < 0 || !std::isfinite(alpha)) return PERF_ERR_SHAPE;
    if (batch > 1 && strideP < (M - 1) * ldp + N) return PERF_ERR_SHAPE;
    const int64_t kLim = INT64_MAX / 8;
    if (M > kLim / lda || N > kLim / ldb || M > kLim / ldp) return PERF_ERR_SHAPE;
    if (batch > 1 && (strideA > kLim / batch || strideB > kLim / batch || strideP > kLim / batch)) return PERF_ERR_SHAPE;
    if (!aligned(A, dtype_size(ab_dt)) || !aligned(B, dtype_size(ab_dt)) || !aligned(P, dtype_size(p_dt)))
        return PERF_ERR_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);

    // One kernel (scores never reach memory): operands as the global->LDS loads need them, N up to 1024, fp32 P for any K
    // that is a multiple of 8 up to 512 (16 x (1024x1024x512): 53 us against 58 in two launches), bf16 P for the K and N that
    // the header names.
    const bool loads_ok = ab_dt == PERF_BF16 && K % 8 == 0 && lda % 8 == 0 && ldb % 8 == 0 && strideA % 8 == 0 && strideB % 8 == 0 &&
                          aligned(A, 16) && aligned(B, 16) && M <= (1 << 24);
    // whole chunks of 128 columns, K = 64 (or what else the LDS holds: 128 x 128, 64 x (512x128x128) 7.0 us against 8.9 with the
    // strip kernel, but 300 x (16x128x128) 7.3 against 5.7), fp32 P with 16-byte aligned rows: B stays in the LDS for several strips, the staged
    // write-out (512 x (512x512x64) 104 us against 116 with the strip kernel, 300 x (256x128x64) 13.2 against 14.5)
    const bool staged = loads_ok && (K == 64 || (K == 128 && N == 128 && M >= 128)) && p_dt == PERF_F32 && lda <= (1 << 21) && ldb <= (1 << 21) && ldp % 4 == 0 &&
                        strideP % 4 == 0 && aligned(P, 16);
    if (staged && N == 512) return launch_fused_staged<32>(A, B, P, M, N, K, lda, ldb, ldp, batch, strideA, strideB, strideP, alpha, st);
    if (staged && N == 256) return launch_fused_staged<16>(A, B, P, M, N, K, lda, ldb, ldp, batch, strideA, strideB, strideP, alpha, st);
    if (staged && N == 128) return launch_fused_staged<8>(A, B, P, M, N, K, lda, ldb, ldp, batch, strideA, strideB, strideP, alpha, st);
    const int64_t strips = (M + 31) / 32 * batch;
    // (5 MiB of fp32 P and less, 4 of bf16: 1 to 8 % ahead; even up to 1.6 times that, with single shapes 7 % behind)
    const bool few = strips * N <= (p_dt == PERF_F32 ? 40960 : 65536);
#define PERF_WIDE(...) return launch_wide<__VA_ARGS__>(A, B, P, M, N, K, lda, ldb, ldp, batch, strideA, strideB, strideP, alpha, st)
    if (loads_ok && lda <= (1 << 21) && ldb <= (1 << 21) && p_dt == PERF_BF16 && N <= 512 && (K == 64 || K == 128)) {
        if (N <= 128 && few) PERF_WIDE(1, uint16_t, 4, false, true);
        if (N <= 128) PERF_WIDE(1, uint16_t, 4);
        if (N <= 256) PERF_WIDE(2, uint16_t, 4);
        // (us, with the four tiles of four waves on their own stages, now: 481 x (32x434x128) 18.6, 16.1, 10 x (679x440x128) 9.1, 7.9;
        // for more than the chip holds at a time 304 x (512x289x128) 82.0, 64.1, 168 x (320x477x64) 26.7, 24.6)
        if (N <= 384 && strips <= 512) PERF_WIDE(3, uint16_t, 4, true);
        if (N <= 384) PERF_WIDE(3, uint16_t, 4);
        if (strips <= 512) PERF_WIDE(2, uint16_t, 8);
        PERF_WIDE(4, uint16_t, 4);
    }
    // A few strips of long rows or long reductions are faster as two launches, which spread the columns over the chip and
    // pipeline deeper (in us, strips on this kernel against two launches): 100x769x128 13 against 8, up to more strips where the
    // GEMM runs its direct kernel on tall tiles (8 x (499x816x64) 12.0 against 11.3); with wider K-ranges from more strips on:
    // 16x200x256 6.8 against 6.4 but 64 x (64x200x256) 7.8 against 8.8, 32x300x384 13.1 against 7.2, 64 x (100x300x384) 16.1
    // against 13.4, 64 x (300x300x512) 30.6 against 46.6, 64 x (16x1024x384) 26 against 21, 64 x (300x1024x384) 59 against 71.
    int64_t least = 0;
    if (N > 512) least = K % 32 == 0 && M >= 64 ? 192 : 64;
    if (K > 128 && N > 128) {
        const int64_t more = N <= 256 ? (K <= 256 ? 96 : 128) : K <= 256 ? 96 : 400;
        least = least > more ? least : more;
    }
    if (loads_ok && lda <= (1 << 20) && ldb <= (1 << 20) && p_dt == PERF_F32 && N <= 1024 && K <= 512 && strips >= least) {
        if (N <= 64 && few) PERF_WIDE(1, float, 2, false, true);
        if (N <= 64) PERF_WIDE(1, float, 2);
        if (N <= 128 && few) PERF_WIDE(1, float, 4, false, true);
        if (N <= 128) PERF_WIDE(1, float, 4);
        if (N <= 256) PERF_WIDE(2, float, 4);
        // Eight waves, or own stages, for what two workgroups per CU hold at a time (512 strips); the shared stages, whose kernels leave
        // room for three and more, for more strips if the reduction is long or the last of the chip's rounds would be nearly
        // empty otherwise.  Us, without these lines, now: 160 x (759x359x384) 145.7, 127.3; 192 x (424x416x512) 137.8, 127.9;
        // 224 x (101x424x16) 14.2, 13.4; 112 x (576x592x384) 116.5, 112.6; 308 x (48x653x8) 16.8, 15.7 (768 strips in one
        // round); 330 x (176x760x192) 100, 89; but 94 x (384x490x72) 25.8 against 27.8, 40 x (514x716x192) 31.4 against 33.2.
        // Four waves with twice the tiles for long reductions of wider rows (242 x (111x800x320) 90, 83; 320 x (32x896x128) 34.5, 31.8;
        // 208 x (224x992x320) 145, 134), and eight for few strips of 513 to 640 columns (64 x (2x616x80) 8.1, 7.8).
        if (N <= 384) {
            if ((strips > 512 && K > 96) || (strips > 256 && K > 256)) PERF_WIDE(3, float, 4);
            PERF_WIDE(3, float, 4, true);
        }
        if (N <= 512) {
            if (strips > 512 && (strips <= 1024 ? K <= 160 : K > 96)) PERF_WIDE(4, float, 4);
            PERF_WIDE(2, float, 8);
        }
        if (N <= 640) {
            if (strips <= 256 && K <= 96) PERF_WIDE(3, float, 8, true);
            if (strips > 768 && K > 256) PERF_WIDE(5, float, 4);
            PERF_WIDE(5, float, 4, true);
        }
        if (N <= 768) {
            if (strips > 512 && (strips <= 768 ? K <= 160 : K > 160)) PERF_WIDE(6, float, 4);
            PERF_WIDE(3, float, 8, true);
        }
        if (strips > 256 && K > (N <= 896 ? 96 : 160)) {
            if (N <= 896) PERF_WIDE(7, float, 4, true);
            PERF_WIDE(8, float, 4, true);
        }
        PERF_WIDE(4, float, 8, true);
    }
#undef PERF_WIDE
    // Unfused: scores into P, then the row softmax in place (fp32 P only).
    if (p_dt != PERF_F32) return PERF_ERR_UNSUPPORTED;
    perf_status s = perf_gemm(A, B, P, M, N, K, PERF_ROW_MAJOR, lda, PERF_COL_MAJOR, ldb, ldp, batch, strideA, strideB,
                              strideP, alpha, ab_dt, PERF_F32, stream);
    if (s != PERF_OK) return s;
    if (batch == 1 || strideP == M * ldp) return perf_softmax(P, P, batch * M, N, ldp, ldp, PERF_F32, PERF_F32, 1.0f, stream);
    for (int64_t b = 0; b < batch; ++b) {
        s = perf_softmax((float *)P + b * strideP, (float *)P + b * strideP, M, N, ldp, ldp, PERF_F32, PERF_F32, 1.0f, stream);
        if (s != PERF_OK) return s;
    }
    return PERF_OK;
}
