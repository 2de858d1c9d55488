"""GPU parity: perf_gemm (MFMA and general kernels) against the CPU oracle.
Tolerance for bf16-input / fp32-accumulate results: max |C^-C| / max(|C|, rms(C)) <= 2e-2,
plus the accumulation-order-independent bound |C^-C| <= K 2^-23 sum_k|a||b|. Exact-integer
problems must match bit for bit."""
import numpy as np
import pytest

import oracle
from workloads import configs, rng
from tests import gpu_helpers as G
from tests import parity as P

pytestmark = pytest.mark.gpu


def _bits(a):
    return rng.f32_to_bf16_bits(np.asarray(a, dtype=np.float32))


def _check(wl, alpha=1.0, c_bf16=False, batch=1, **kw):
    d = wl.make()
    a, b = d["a_bf16"], d["b_bf16"]
    if batch > 1:
        a = np.stack([np.roll(a, i, axis=0) for i in range(batch)])
        b = np.stack([np.roll(b, -i, axis=1) for i in range(batch)])
    c = G.run_gemm(a, b, wl.M, wl.N, wl.K, alpha=alpha, batch=batch, c_bf16=c_bf16, **kw)
    ad, bd = oracle.widen(a, bf16=True), oracle.widen(b, bf16=True)
    ref = oracle.gemm(ad, bd, wl.M, wl.N, wl.K, b_col=True, alpha=float(np.float32(alpha)), batch=batch)
    ref = ref.reshape(batch, wl.M, wl.N)
    for i in range(batch):
        ai = ad.reshape(batch, -1)[i]
        bi = bd.reshape(batch, -1)[i]
        s = abs(float(np.float32(alpha))) * oracle.gemm_absdot(ai, bi, wl.M, wl.N, wl.K, b_col=True)
        ci = P.bf16_to_f64(c[i]) if c_bf16 else c[i]
        P.assert_contraction_close(ci, ref[i], s, wl.K, out_bf16=c_bf16)


@pytest.mark.parametrize("M,N,K", [
    (256, 256, 64), (128, 128, 128), (256, 512, 256), (300, 200, 192), (1, 1, 64), (257, 129, 128),
    (64, 640, 64), (33, 7, 512), (768, 1024, 1024), (512, 512, 64),
])
def test_mfma_path_shapes_and_tails(M, N, K):
    _check(configs.GemmWorkload(M=M, N=N, K=K))


def test_mfma_large_tile_path_with_tails():
    # enough 256x256 tiles to select the 4x4-wave-tile kernel, with ragged M and N
    _check(configs.GemmWorkload(M=4096 - 37, N=4096 + 19, K=128))


def test_alpha_bf16_output_batched_and_padded_ld():
    _check(configs.GemmWorkload(M=160, N=96, K=128), alpha=0.125)
    _check(configs.GemmWorkload(M=160, N=96, K=128), c_bf16=True)
    _check(configs.GemmWorkload(M=130, N=70, K=64), alpha=0.125, batch=5)
    wl = configs.GemmWorkload(M=96, N=80, K=64)
    d = wl.make()
    a = np.zeros((96, 72), np.uint16); a[:, :64] = d["a_bf16"]
    b = np.zeros((80, 88), np.uint16); b[:, :64] = d["b_bf16"]
    c = G.run_gemm(a, b, 96, 80, 64, lda=72, ldb=88, ldc=84)[0]
    ref = oracle.gemm(oracle.widen(d["a_bf16"], True), oracle.widen(d["b_bf16"], True), 96, 80, 64, b_col=True)
    s = oracle.gemm_absdot(oracle.widen(d["a_bf16"], True), oracle.widen(d["b_bf16"], True), 96, 80, 64, b_col=True)
    P.assert_contraction_close(c, ref, s, 64)


def test_mid_tile_kernels():
    # 128x128 tiles are chosen between 192 such tiles and 256 tiles of 256x256; smaller problems get 64x64 tiles
    _check(configs.GemmWorkload(M=1792, N=1800, K=64))      # K-step-32 loop, 128x128 tiles, ragged N
    _check(configs.GemmWorkload(M=1792, N=1792, K=512))     # 128x128 tiles, long reduction
    _check(configs.GemmWorkload(M=1792, N=1792, K=512), tile=128, kstep=64)


def test_k64_loop_tails_alpha_bf16_batched_and_odd_ldc():
    # the K-step-64 loop (16x16x32 MFMAs, lane-exchange epilogue, bf16 C staged through LDS); the
    # library picks it for 256x256 tiles with K a multiple of 64 and >= 512, the smaller tiles are named
    _check(configs.GemmWorkload(M=300, N=200, K=576), tile=128, kstep=64)      # ragged, odd step count
    _check(configs.GemmWorkload(M=256, N=384, K=512), alpha=0.125, tile=128, kstep=64)  # full tiles, vector epilogue, alpha
    _check(configs.GemmWorkload(M=256, N=256, K=512), c_bf16=True, tile=128, kstep=64)  # bf16 epilogue through LDS
    _check(configs.GemmWorkload(M=256, N=256, K=512), c_bf16=True, tile=64, kstep=64)
    _check(configs.GemmWorkload(M=512, N=256, K=128), c_bf16=True, tile=256, kstep=64)
    _check(configs.GemmWorkload(M=130, N=70, K=512), alpha=-2.0, batch=3, c_bf16=True, tile=128, kstep=64)
    _check(configs.GemmWorkload(M=130, N=70, K=512), alpha=-2.0, batch=3, c_bf16=True, tile=64, kstep=64)
    _check(configs.GemmWorkload(M=512, N=512, K=512), batch=64)                # 256 tiles of 256x256: the large-tile kernel
    _check(configs.GemmWorkload(M=512, N=512, K=512), batch=64, c_bf16=True)
    _check(configs.GemmWorkload(M=2048 + 40, N=2048 - 24, K=640))              # large-tile kernel with ragged edges
    wl = configs.GemmWorkload(M=256, N=256, K=512)
    d = wl.make()
    c = G.run_gemm(d["a_bf16"], d["b_bf16"], 256, 256, 512, ldc=258, tile=128, kstep=64)[0]  # ldc not a multiple of 4: scalar epilogue
    ad, bd = oracle.widen(d["a_bf16"], True), oracle.widen(d["b_bf16"], True)
    ref = oracle.gemm(ad, bd, 256, 256, 512, b_col=True)
    P.assert_contraction_close(c, ref, oracle.gemm_absdot(ad, bd, 256, 256, 512, b_col=True), 512)

@pytest.mark.gpu
def test_k64_loop_with_32x32_mfma():
    """The K-step-64 loop of the 256x256 tile built on the 32x32x16 MFMA: ragged edges, several k-steps, alpha, batch, bf16 C."""
    _check(configs.GemmWorkload(M=512, N=256, K=128), tile=256, kstep=65)
    _check(configs.GemmWorkload(M=300, N=520, K=576), tile=256, kstep=65, alpha=0.25)
    _check(configs.GemmWorkload(M=258, N=130, K=64), tile=256, kstep=65, batch=2, c_bf16=True)
    _check(configs.GemmWorkload(M=1024, N=768, K=1024), tile=256, kstep=65, c_bf16=True)



def test_deep_ring_loop():
    # K-step-32 loop with the ring filling the LDS (16 stages of a 64x64 tile, 8 of a 128x128 one):
    # reductions shorter than, equal to and longer than the ring, ragged tiles, batches, bf16 C
    for tile in (64, 128):
        _check(configs.GemmWorkload(M=100, N=70, K=64), tile=tile, kstep=33)
        _check(configs.GemmWorkload(M=192, N=130, K=512), tile=tile, kstep=33, alpha=0.5)
        _check(configs.GemmWorkload(M=130, N=260, K=1056), tile=tile, kstep=33, batch=2, c_bf16=True)
    _check(configs.GemmWorkload(M=512, N=512, K=2048))      # one round of 64x64 tiles, long reduction: the library's own choice


@pytest.mark.parametrize("a_col,b_col", [(False, False), (True, False), (True, True), (False, True)])
@pytest.mark.parametrize("M,N,K", [(5, 7, 3), (65, 63, 17), (100, 130, 65)])
def test_general_kernel_layouts_exact_integers(a_col, b_col, M, N, K):
    g = np.random.default_rng(M + N + K)
    a = g.integers(-8, 9, (M, K)).astype(np.float32)
    b = g.integers(-8, 9, (K, N)).astype(np.float32)
    a_st = a.T.copy() if a_col else a
    b_st = b.T.copy() if b_col else b
    ref = oracle.gemm(a_st, b_st, M, N, K, a_col=a_col, b_col=b_col, alpha=0.5)
    c16 = G.run_gemm(_bits(a_st), _bits(b_st), M, N, K, a_col=a_col, b_col=b_col, alpha=0.5)[0]
    c32 = G.run_gemm(a_st, b_st, M, N, K, a_col=a_col, b_col=b_col, alpha=0.5, ab_bf16=False)[0]
    assert np.array_equal(c16.astype(np.float64), ref) and np.array_equal(c32.astype(np.float64), ref)


@pytest.mark.parametrize("ab_bf16,c_bf16", [(True, False), (True, True), (False, False)])
@pytest.mark.parametrize("a_col,b_col", [(False, False), (True, False), (True, True), (False, True)])
@pytest.mark.parametrize("M,N,K,batch,pad", [
    (1, 1, 1, 1, 0), (7, 3, 5, 2, 0), (3, 300, 7, 1, 1),       # extents below a 16-byte load: element loads
    (8, 9, 8, 1, 0), (64, 64, 64, 1, 0), (65, 71, 130, 2, 3),    # one tile; exact, ragged in every extent, odd ld (the waves' kernel)
    (100, 70, 643, 1, 1), (64, 130, 1024, 1, 0), (9, 10, 257, 3, 1),   # long reductions on few tiles (the waves' kernel)
    (64, 72, 704, 1, 0), (72, 64, 288, 1, 0), (64, 64, 1216, 1, 0),
    (705, 741, 577, 1, 1), (704, 744, 704, 1, 0), (704, 744, 1088, 1, 0),   # two groups of waves (bf16, row-major): K-steps that they
                                                                 # do not divide, with edges and without
    (70, 65, 96, 65, 1), (100, 66, 67, 100, 0),                  # 64 x 64 (fp32), one register set
    (64, 61, 300, 641, 0),                                       # ... four
    (257, 131, 97, 64, 0), (130, 250, 64, 96, 5),                # 128 x 128 (bf16), 256 x 128 (fp32)
    (40, 33, 521, 200, 1), (300, 261, 512, 100, 0),              # 256 x 256 (bf16): ragged first and second tiles
    (500, 250, 70, 40, 1), (128, 120, 65, 130, 0), (33, 65, 20, 128, 0),   # 256 x 128 (fp32), full and half full; 64 x 64 instead
    (3, 70, 40, 2, 1), (70, 2, 20, 3, 0), (1, 9, 8, 1, 0),       # element loads for the short operand only
    (3, 70, 130, 2, 1), (70, 2, 77, 3, 0),                       # ... short operands of the waves' kernel
    (70, 130, 40, 1, 1), (70, 130, 31, 1, 0),                    # one register set for short reductions (bf16, fp32)
    (70, 130, 64, 1, 1), (70, 130, 65, 1, 0), (70, 130, 97, 1, 0),   # ... of the waves' kernel
])
def test_staged_kernel_edges(M, N, K, batch, pad, a_col, b_col, ab_bf16, c_bf16):
    """Every layout and type of the register-staged contraction at the edges of its tiles, K-steps and loads."""
    g = np.random.default_rng(M * 1000 + N + K)
    lda, ldb = (M if a_col else K) + pad, (K if b_col else N) + pad
    a = g.uniform(-1, 1, (batch, K if a_col else M, lda)).astype(np.float32)
    b = g.uniform(-1, 1, (batch, N if b_col else K, ldb)).astype(np.float32)
    if ab_bf16:
        a, b = _bits(a), _bits(b)
    c = G.run_gemm(a, b, M, N, K, a_col=a_col, b_col=b_col, batch=batch, ab_bf16=ab_bf16, c_bf16=c_bf16, lda=lda, ldb=ldb,
                   ldc=N + pad, alpha=0.75)
    for i in sorted({0, batch // 2, batch - 1}):
        ai, bi = oracle.widen(a[i], ab_bf16), oracle.widen(b[i], ab_bf16)
        ref = oracle.gemm(ai, bi, M, N, K, a_col=a_col, b_col=b_col, alpha=0.75, lda=lda, ldb=ldb)
        A = ai[:, :M].T if a_col else ai[:, :K]
        B = bi[:, :K].T if b_col else bi[:, :N]
        absdot = 0.75 * (np.abs(A) @ np.abs(B))
        # fp32 operands: the products that the split leaves out are at most 2^-24 of |a||b| each (K + 1 in the bound)
        P.assert_contraction_close(P.bf16_to_f64(c[i]) if c_bf16 else c[i], ref, absdot, K + 1, out_bf16=c_bf16)


@pytest.mark.parametrize("ab_bf16,c_bf16", [(True, False), (True, True), (False, False)])
@pytest.mark.parametrize("a_col,b_col", [(False, False), (True, False), (True, True), (False, True)])
@pytest.mark.parametrize("M,N,K,batch,pad", [
    (1, 1, 64, 1, 0), (33, 65, 65, 2, 1), (5, 7, 1031, 1, 0),    # 32 x 32: one K-step, the last one overlapping, more than waves
    (64, 64, 512, 1, 0), (31, 97, 8 * 64 + 1, 3, 3),             # ... the last step alone in its round; the direct kernels' shapes
    (33, 65, 32, 1, 0), (33, 65, 63, 3, 1),                      # fp32: one K-step, one and most of another
    (700, 600, 40, 1, 1), (577, 450, 66, 1, 0),                  # 32 x 32 with four waves (fp32), pairs of tiles (bf16); an odd row alone
    (450, 577, 127, 1, 1), (450, 577, 513, 1, 1),                # in the last pair, an odd column (row-major)
    (705, 641, 1030, 1, 0),                                      # ... the longest of a few tiles; 64 x 64 with eight waves (fp32)
    (20, 9000, 130, 1, 1), (9000, 20, 513, 1, 0),                # pairs along the only operand with more than a tile
    (705, 741, 64, 1, 1), (705, 741, 100, 1, 0), (705, 741, 128, 1, 1),   # two waves: one K-step, the last overlapping, one each
    (705, 741, 200, 1, 1), (705, 741, 400, 1, 0),                # one round of 64 x 64: 32 x 32 and pairs
    (705, 741, 1030, 1, 0), (705, 741, 2113, 1, 1), (768, 768, 2080, 1, 0),   # ... 64 x 64 with eight waves; the direct kernels' shapes
    (1030, 1090, 70, 1, 0), (1030, 1090, 130, 1, 1), (1030, 1090, 300, 1, 1),   # several rounds: two waves; pairs with two and four
    (1025, 1089, 515, 1, 0), (1025, 1089, 1100, 1, 1),           # ... 64 x 64, ragged by one
    (100, 70, 130, 37, 3), (65, 33, 200, 11, 0), (64, 64, 520, 300, 0),   # batches that 8 does not divide, tiles that it does not
])
def test_waves_kernel_edges(M, N, K, batch, pad, a_col, b_col, ab_bf16, c_bf16):
    """Every layout and type of the contraction whose waves divide K, at the edges of its tiles, K-steps and row pairs (the
    smallest K of each type included); padding of C stays as it was."""
    test_staged_kernel_edges(M, N, K, batch, pad, a_col, b_col, ab_bf16, c_bf16)


@pytest.mark.parametrize("a_col,b_col", [(False, False), (True, True)])
@pytest.mark.parametrize("M,N,K,batch", [(70, 65, 33, 1), (96, 64, 300, 1), (130, 250, 64, 96), (7, 3, 5, 1),
                                         (70, 65, 33, 65), (64, 61, 100, 641)])   # (the staged kernel's 64 x 64)
def test_fp32_range_ends(M, N, K, batch, a_col, b_col):
    """fp32 operands at both ends of the range: values around 2^-118 (below what the three-way split holds), one of
    them among ordinary ones, and values next to the largest. Bounds as for any fp32 accumulation order."""
    g = np.random.default_rng(K)
    for scale, where in ((2.0 ** -118, None), (2.0 ** -118, 3), (1.9 * 2.0 ** 126, None)):
        a = g.uniform(0.5, 1, (batch, K, M) if a_col else (batch, M, K))
        b = g.uniform(0.5, 1, (batch, N, K) if b_col else (batch, K, N)) / (1 if where is None and scale < 1 else 4 * K)
        if where is None:
            a = a * scale
        else:
            a.reshape(batch, -1)[:, where] *= scale
        a, b = a.astype(np.float32), b.astype(np.float32)
        c = G.run_gemm(a, b, M, N, K, a_col=a_col, b_col=b_col, batch=batch, ab_bf16=False)
        for i in (0, batch - 1):
            ref = oracle.gemm(a[i], b[i], M, N, K, a_col=a_col, b_col=b_col)
            P.assert_contraction_close(c[i], ref, oracle.gemm_absdot(a[i], b[i], M, N, K, a_col=a_col, b_col=b_col), K + 1)


def split_bound(K):
    """Largest error over sum |a||b| of an fp32 reduction of K: K roundings of the partial sum with the fp32 instruction
    (K < 8); else the products that the three-way split leaves out (2^-24 each) and, for every 16 k, six additions to
    the accumulator that may truncate, of which in the first 16 only the last is to more than 2^-7 of the sum."""
    return K * 2.0 ** -24 if K < 8 else 2.0 ** -24 + (1.04 + 6 * ((K + 15) // 16 - 1)) * 2.0 ** -23


@pytest.mark.parametrize("a_col,b_col", [(False, True), (True, False), (False, False)])
@pytest.mark.parametrize("K", [1, 2, 7, 8, 16, 33, 300, 4096])
def test_fp32_operands_that_split_badly(K, a_col, b_col):
    """fp32 operands whose lower parts are as large as they get for splits by truncation (1 + 2^-7 - 2^-23) and by rounding
    (1 + 2^-8 - 2^-17), all of one sign: what a split leaves out adds up."""
    M, N = 70, 130
    g = np.random.default_rng(K)
    adv = np.array([1 + 2.0 ** -7 - 2.0 ** -23, 1 + 2.0 ** -8 - 2.0 ** -17 - 2.0 ** -23, 1 + 2.0 ** -8 + 2.0 ** -17, 1.0])
    for a, b in ((np.full((M, K), adv[0]), np.full((N, K), adv[0])), (adv[g.integers(0, 4, (M, K))], adv[g.integers(0, 4, (N, K))]),
                 (g.uniform(0.5, 1, (M, K)), g.uniform(0.5, 1, (N, K)))):
        a, b = a.astype(np.float32), b.astype(np.float32)
        c = G.run_gemm(np.ascontiguousarray(a.T) if a_col else a, b if b_col else np.ascontiguousarray(b.T), M, N, K, a_col=a_col,
                       b_col=b_col, ab_bf16=False)[0]
        ref = a.astype(np.float64) @ b.astype(np.float64).T
        rel = np.abs(c - ref) / ref
        assert rel.max() <= split_bound(K), rel.max()
        if K >= 16 and a.min() < 1:  # random operands: the additions' errors are independent
            assert np.sqrt(np.mean(rel ** 2)) <= 2.0 ** -24 * np.sqrt(6 * K / 16)


@pytest.mark.parametrize("a_col,b_col", [(False, True), (True, False)])
@pytest.mark.parametrize("M,N,K", [(70, 65, 33), (96, 64, 300), (7, 3, 5), (3, 9, 40)])
def test_fp32_values_next_to_what_splits(M, N, K, a_col, b_col):
    """Values whose lowest part just fits a bf16 (2^-109), values that round to infinity in one (next to FLT_MAX), and infinities
    and NaN, which the fp32 instruction carries through."""
    g = np.random.default_rng(M)
    big = np.float32(np.finfo(np.float32).max)
    run = lambda a, b: G.run_gemm(np.ascontiguousarray(a.T) if a_col else a, b if b_col else np.ascontiguousarray(b.T), M, N, K,  # noqa: E731
                                  a_col=a_col, b_col=b_col, ab_bf16=False)[0]
    a0, b = g.uniform(0.5, 1, (M, K)).astype(np.float32), g.uniform(0.5, 1, (N, K)).astype(np.float32)
    for scale, at, value in ((2.0 ** -109, None, 0), (1, (2, 4), big), (1, (2, 4), -big)):
        a = a0 * np.float32(scale)
        if at is not None:
            a[at] = value
        ref, ab = a.astype(np.float64) @ b.astype(np.float64).T / K, np.abs(a).astype(np.float64) @ b.astype(np.float64).T / K
        # (the added 2^-126: half the smallest subnormal per addition)
        P.assert_contraction_close(run(a, b / np.float32(K)), ref, ab + 2.0 ** -126, K + 2)
    for value in (np.inf, -np.inf, np.nan):
        a = a0.copy()
        a[2, 4] = value
        c = run(a, b)
        assert np.all(np.isnan(c[2])) if np.isnan(value) else np.all(c[2] == value)
        rest = np.arange(M) != 2
        ref = a0.astype(np.float64) @ b.astype(np.float64).T
        P.assert_contraction_close(c[rest], ref[rest], ref[rest], K + 1)


@pytest.mark.parametrize("a_col,b_col", [(False, True), (True, False)])
@pytest.mark.parametrize("M,N,K,batch", [(70, 65, 33, 1), (64, 64, 96, 1), (96, 64, 300, 1), (130, 250, 64, 96), (3, 9, 40, 1),
                                         (70, 65, 33, 65), (64, 61, 100, 641)])   # (the staged kernel's 64 x 64)
def test_fp32_tiny_values(M, N, K, batch, a_col, b_col):
    """Values under 2^-110 (which need more than the three-way split): beside ordinary ones in sums that they do not
    show in, alone in the sums of some columns, in both operands, and beside values that leave no room to scale."""
    g = np.random.default_rng(M + K)
    t = 2.0 ** -112
    a0, b0 = g.uniform(0.5, 1, (M, K)), g.uniform(0.5, 1, (N, K))
    beside, alone = a0.copy(), b0.copy()
    beside[:, ::2] *= t
    alone[N // 2:, 1::2] = 0                 # the second half of the columns meets tiny values only
    room = beside.copy()
    room[0, 1] = 2.0 ** 120
    for a, b in ((beside, b0), (beside, alone), (a0 * t, b0), (beside, b0 * np.where(np.arange(K) % 3, 1.0, t)), (room, alone),
                 (a0, beside[:1] * np.ones((N, 1)))):
        a, b = a.astype(np.float32), b.astype(np.float32)
        A, B = np.ascontiguousarray(a.T) if a_col else a, b if b_col else np.ascontiguousarray(b.T)
        c = G.run_gemm(np.tile(A, (batch, 1)), np.tile(B, (batch, 1)), M, N, K, a_col=a_col, b_col=b_col, batch=batch, ab_bf16=False)
        ref = a.astype(np.float64) @ b.astype(np.float64).T
        for i in (0, batch - 1):
            # (the added 2^-126: half the smallest subnormal per addition)
            P.assert_contraction_close(c[i], ref, ref + 2.0 ** -126, K + 1)
            rel = np.abs(c[i] - ref) / np.maximum(ref, K * 2.0 ** -126)
            assert rel.max() <= (K + 1) * 2.0 ** -23


@pytest.mark.parametrize("M,N,K,tiny_row,tiny_col", [(70, 70, 300, 5, None), (70, 70, 300, None, 5), (65, 131, 33, 3, 66),
                                                     (257, 129, 40, None, 128), (199, 67, 1024, 130, 65)])
def test_rows_shared_by_two_tiles_have_one_writer(M, N, K, tiny_row, tiny_col):
    """K-strided fp32 operands with ragged last tiles and a value under 2^-110 in some tiles only (those may take another way):
    every element carries the bits of the 64 x 64 tile that owns it, in every run. A tile's bits alone come from a call on its
    rows and columns. (These shapes run the contraction whose waves divide K, the staged one's are below.)"""
    g = np.random.default_rng(M + N)
    a, b = g.uniform(-1, 1, (K, M)).astype(np.float32), g.uniform(-1, 1, (K, N)).astype(np.float32)
    if tiny_row is not None:
        a[7, tiny_row] = 1.7 * 2.0 ** -118
    if tiny_col is not None:
        b[9, tiny_col] = 1.7 * 2.0 ** -118
    c = G.run_gemm(a, b, M, N, K, a_col=True, b_col=False, ab_bf16=False)[0]
    for _ in range(5):
        assert np.array_equal(c, G.run_gemm(a, b, M, N, K, a_col=True, b_col=False, ab_bf16=False)[0])
    for m0 in range(0, M, 64):
        for n0 in range(0, N, 64):
            m1, n1 = min(M, m0 + 64), min(N, n0 + 64)
            m, n = m0 - (m0 - m1) % 4, n0 - (n0 - n1) % 4  # (the tile reads whole blocks of 4)
            own = G.run_gemm(a[:, m:m1], b[:, n:n1], m1 - m, n1 - n, K, a_col=True, b_col=False, ab_bf16=False)[0]
            assert np.array_equal(c[m0:m1, n0:n1], own[m0 - m:, n0 - n:])


@pytest.mark.parametrize("M,N,K,tiny_row,tiny_col", [(1061, 1030, 40, 1040, None), (1061, 1030, 96, None, 1026), (1633, 1630, 130, 1605, 1626)])
def test_rows_shared_by_two_tiles_have_one_writer_staged(M, N, K, tiny_row, tiny_col):
    """As above on shapes that the staged kernel runs, with 64 x 64 tiles: there a ragged last tile starts early and reads rows
    and columns that its neighbour stores. A tile's bits alone come from a batch of it that the same kernel runs."""
    g = np.random.default_rng(M + N)
    a, b = g.uniform(-1, 1, (K, M)).astype(np.float32), g.uniform(-1, 1, (K, N)).astype(np.float32)
    if tiny_row is not None:
        a[7, tiny_row] = 1.7 * 2.0 ** -118
    if tiny_col is not None:
        b[9, tiny_col] = 1.7 * 2.0 ** -118
    c = G.run_gemm(a, b, M, N, K, a_col=True, b_col=False, ab_bf16=False)[0]
    for _ in range(3):
        assert np.array_equal(c, G.run_gemm(a, b, M, N, K, a_col=True, b_col=False, ab_bf16=False)[0])
    ref = a.T.astype(np.float64) @ b.astype(np.float64)
    P.assert_contraction_close(c, ref, np.abs(a).T.astype(np.float64) @ np.abs(b).astype(np.float64), K + 1)
    last_m, last_n, copies = (M - 1) // 64 * 64, (N - 1) // 64 * 64, 641
    for m0 in (last_m - 64, last_m):
        for n0 in (last_n - 64, last_n):
            m1, n1 = min(M, m0 + 64), min(N, n0 + 64)
            m, n = m0 - (m0 - m1) % 4, n0 - (n0 - n1) % 4  # (the tile reads whole blocks of 4)
            own = G.run_gemm(np.tile(a[:, m:m1], (copies, 1)), np.tile(b[:, n:n1], (copies, 1)), m1 - m, n1 - n, K, a_col=True, b_col=False,
                             batch=copies, ab_bf16=False)
            for i in (0, copies - 1):
                assert np.array_equal(c[m0:m1, n0:n1], own[i][m0 - m:, n0 - n:])


def test_mfma_exact_integers_identity_permutation_ones():
    g = np.random.default_rng(3)
    M, N, K = 200, 136, 192
    a = g.integers(-8, 9, (M, K)).astype(np.float32)
    bs = g.integers(-8, 9, (N, K)).astype(np.float32)           # column-major storage of B
    ref = oracle.gemm(a, bs, M, N, K, b_col=True)
    assert np.array_equal(G.run_gemm(_bits(a), _bits(bs), M, N, K)[0].astype(np.float64), ref)
    n = 128
    a = rng.bf16_bits_to_f32(configs.GemmWorkload(M=n, N=n, K=n).make()["a_bf16"])
    eye = np.eye(n, dtype=np.float32)
    assert np.array_equal(G.run_gemm(_bits(a), _bits(eye), n, n, n)[0], a)            # B = I
    assert np.array_equal(G.run_gemm(_bits(eye), _bits(a), n, n, n)[0], a.T)          # A = I: C = B = storage^T
    # cyclic shift: B[k][n] = [k == (n+1) mod K]; stored column-major => bs[n][k]
    bs = np.zeros((n, n), np.float32)
    for col in range(n):
        bs[col, (col + 1) % n] = 1.0
    assert np.array_equal(G.run_gemm(_bits(a), _bits(bs), n, n, n)[0], np.roll(a, -1, axis=1))
    ones = G.run_gemm(_bits(np.ones((70, 320))), _bits(np.ones((90, 320))), 70, 90, 320)[0]
    assert np.array_equal(ones, np.full((70, 90), 320.0, np.float32))


@pytest.mark.parametrize("tile,kstep", [(0, 0), (256, 65)])
def test_config3_full_size_sampled_rows(tile, kstep):
    """4096^3 in the benchmark's launch configuration (and with the 32x32x16 variant of its main
    loop); 48 sampled rows of C (all columns) are recomputed by the oracle, and the whole C is
    checked against row/column sums."""
    wl = configs.CONFIG3
    d = wl.make()
    c = G.run_gemm(d["a_bf16"], d["b_bf16"], wl.M, wl.N, wl.K, tile=tile, kstep=kstep)[0]
    rows = np.unique(np.concatenate([np.arange(0, wl.M, 89), [255, 256, 4095]]))
    a_s = oracle.widen(d["a_bf16"][rows], True)
    bd = oracle.widen(d["b_bf16"], True)
    ref = oracle.gemm(a_s, bd, len(rows), wl.N, wl.K, b_col=True)
    s = oracle.gemm_absdot(a_s, bd, len(rows), wl.N, wl.K, b_col=True)
    P.assert_contraction_close(c[rows], ref, s, wl.K)
    # property over every entry: C @ 1 = A @ (B @ 1), in float64 (tolerance: fp32 accumulation
    # error of one entry, <= K 2^-23 sum|a||b| <= K^2 2^-23, times sqrt(N) for the sum)
    af = oracle.widen(d["a_bf16"], True)
    rowsum_ref = af @ bd.sum(axis=0)
    assert np.max(np.abs(c.astype(np.float64).sum(axis=1) - rowsum_ref)) < 1.0


@pytest.mark.parametrize("c_bf16", [False, True])
def test_config3_full_size_every_entry_exact_integers(c_bf16):
    """4096^3 in the benchmark's launch configuration with small-integer operands (|v| <= 8): every
    product and every partial sum is an integer below 2^24, exact in fp32 whatever the order, so
    all 16.7M entries of C must equal the exact product bit for bit. The exact product is a float64
    matmul on the host (exact for the same reason), tied to the oracle on sampled rows. With bf16 C
    the expected bits are the oracle's single rounding of the exact value."""
    wl = configs.CONFIG3
    g = np.random.default_rng(303)
    a = g.integers(-8, 9, (wl.M, wl.K)).astype(np.float32)
    bs = g.integers(-8, 9, (wl.N, wl.K)).astype(np.float32)      # column-major storage of B
    exact = a.astype(np.float64) @ bs.astype(np.float64).T
    rows = np.array([0, 255, 256, 1777, 4095])
    assert np.array_equal(oracle.gemm(a[rows].astype(np.float64), bs.astype(np.float64), len(rows), wl.N, wl.K, b_col=True),
                          exact[rows])
    c = G.run_gemm(_bits(a), _bits(bs), wl.M, wl.N, wl.K, c_bf16=c_bf16)[0]
    if c_bf16:
        assert np.array_equal(c, oracle.round_bf16(exact))
    else:
        assert np.array_equal(c.astype(np.float64), exact)


def test_config4_attention_scores_then_softmax():
    """Q K^T / 8 for 512 (batch x head) matrices, then row softmax of the 262144 x 512
    scores: all batches on the GPU; three batches recomputed by the oracle."""
    import torch
    import paper_2511_03586_amd as perf
    wl = configs.CONFIG4
    d = wl.make()
    qd, kd = G.dev(d["q_bf16"]), G.dev(d["k_bf16"])
    S, D, B = wl.seq, wl.d, wl.batch
    sd = torch.empty(B * S * S, dtype=torch.float32, device="cuda")
    pd = torch.empty_like(sd)
    perf.perf_gemm(qd.data_ptr(), kd.data_ptr(), sd.data_ptr(), S, S, D, perf.PERF_ROW_MAJOR, D,
                   perf.PERF_COL_MAJOR, D, S, B, S * D, S * D, S * S, wl.alpha, perf.PERF_BF16, perf.PERF_F32,
                   G.stream())
    perf.perf_softmax(sd.data_ptr(), pd.data_ptr(), B * S, S, S, S, perf.PERF_F32, perf.PERF_F32, 1.0, G.stream())
    torch.cuda.synchronize()
    assert float((pd.view(B * S, S).double().sum(dim=1) - 1.0).abs().max()) < 1e-5
    for b in (0, 257, 511):
        q, k = oracle.widen(d["q_bf16"][b], True), oracle.widen(d["k_bf16"][b], True)
        s_ref = oracle.gemm(q, k, S, S, D, b_col=True, alpha=wl.alpha)
        absdot = wl.alpha * oracle.gemm_absdot(q, k, S, S, D, b_col=True)
        s_gpu = sd.view(B, S, S)[b].cpu().numpy()
        P.assert_contraction_close(s_gpu, s_ref, absdot, D)
        p_gpu = pd.view(B, S, S)[b].cpu().numpy()
        P.assert_softmax_close(p_gpu, oracle.softmax(s_ref))
        # argmax exact on rows the oracle can decide (top-two scores more than 1e-5 apart)
        top2 = np.sort(s_ref, axis=1)[:, -2:]
        decidable = (top2[:, 1] - top2[:, 0]) > 1e-5
        assert np.array_equal(p_gpu.argmax(axis=1)[decidable], s_ref.argmax(axis=1)[decidable])


def test_deterministic():
    d = configs.GemmWorkload(M=512, N=512, K=512).make()
    c0 = G.run_gemm(d["a_bf16"], d["b_bf16"], 512, 512, 512)
    c1 = G.run_gemm(d["a_bf16"], d["b_bf16"], 512, 512, 512)
    assert np.array_equal(c0, c1)


def test_more_tiles_than_a_launch_holds():
    """2^24 tiles and more of 256 threads (a dimension of 2^32 threads is cut short without an error): B one value."""
    import torch
    import paper_2511_03586_amd as perf
    big = (1 << 30) + 5
    x = torch.zeros(big, dtype=torch.bfloat16, device="cuda")
    x[::1 << 20] = 3.0
    x[-1] = 5.0
    one = torch.full((8,), 2.0, dtype=torch.bfloat16, device="cuda")
    c = torch.full((big,), 7.0, dtype=torch.bfloat16, device="cuda")
    perf.perf_gemm(x.data_ptr(), one.data_ptr(), c.data_ptr(), big, 1, 1, perf.PERF_ROW_MAJOR, 1, perf.PERF_COL_MAJOR, 1, 1, 1, 0, 0, 0,
                   1.0, perf.PERF_BF16, perf.PERF_BF16, G.stream())
    assert bool((c == 2.0 * x).all())
