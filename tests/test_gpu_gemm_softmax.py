"""GPU parity: perf_gemm_softmax (fused kernel and the two-operator path) against the CPU oracle.
Gate: the bar for fp32 reductions, max relative error 1e-5 over probabilities >= 1e-30 (absolute
1e-35 below), bf16 results one bf16 rounding (2^-8) more. The measured worst error of every case
is printed (run pytest with -s to see it); the accumulation-order bound K 2^-24 |alpha| max sum|a||b|
on the scores is printed beside it for comparison only, it is not the gate."""
import numpy as np
import pytest

import oracle
from workloads import configs, rng
from tests import gpu_helpers as G
from tests import parity as P

pytestmark = pytest.mark.gpu


def _inputs(M, N, K, batch, seed=0, sigma=1.0):
    q = rng.normal(rng.tensor_seed(4, 0, seed), (batch, M, K), 0.0, sigma)
    k = rng.normal(rng.tensor_seed(4, 1, seed), (batch, N, K), 0.0, sigma)
    return rng.f32_to_bf16_bits(q), rng.f32_to_bf16_bits(k)


TOL = 1e-5


def _score_bound(ad, bd, M, N, K, alpha, batch):
    worst = 0.0
    for i in range(batch):
        s = oracle.gemm_absdot(ad.reshape(batch, -1)[i], bd.reshape(batch, -1)[i], M, N, K, b_col=True)
        worst = max(worst, float(s.max()))
    return K * 2.0 ** -24 * abs(alpha) * worst


def _check(M, N, K, alpha=0.125, batch=1, p_bf16=False, seed=0, **kw):
    a, b = _inputs(M, N, K, batch, seed)
    p = G.run_gemm_softmax(a, b, M, N, K, alpha=alpha, batch=batch, p_bf16=p_bf16, **kw)
    ad, bd = oracle.widen(a, True), oracle.widen(b, True)
    ref = oracle.gemm_softmax(ad, bd, M, N, K, alpha=float(np.float32(alpha)), batch=batch)
    if p_bf16:
        got = P.bf16_to_f64(p)
        err = float(np.max(np.abs(got - ref) / np.maximum(ref, 2.0 ** -20)))
        print(f"gemm_softmax {M}x{N}x{K} batch {batch} alpha {alpha} bf16 P: max rel err {err:.3e}")
        assert err <= 2.0 ** -8 + TOL
    else:
        rel, _ = P.softmax_max_rel_err(p.reshape(-1, N), ref.reshape(-1, N))
        print(f"gemm_softmax {M}x{N}x{K} batch {batch} alpha {alpha}: max rel err {rel:.3e} "
              f"(score-order bound {_score_bound(ad, bd, M, N, K, float(np.float32(alpha)), batch):.3e})")
        P.assert_softmax_close(p.reshape(-1, N), ref.reshape(-1, N), tol=TOL)
        np.testing.assert_allclose(p.astype(np.float64).sum(-1), 1.0, atol=1e-5)
    return p, ref


@pytest.mark.parametrize("M,N,K", [
    (128, 512, 64), (512, 512, 64), (300, 500, 64), (1, 1, 32), (37, 64, 32), (129, 65, 96),
    (256, 128, 128), (200, 256, 128), (64, 257, 64), (5, 33, 32),
])
def test_fused_kernel_shapes_tails_and_masks(M, N, K):
    _check(M, N, K)


def test_fused_alpha_signs_batches_bf16_output_and_padded_ld():
    _check(160, 512, 64, alpha=-0.125)
    _check(160, 192, 64, alpha=0.0)          # all scores equal: every probability 1/N
    _check(130, 70, 64, alpha=0.5, batch=5)
    _check(256, 512, 64, p_bf16=True)
    _check(100, 300, 64, p_bf16=True, batch=2)
    M, N, K = 96, 80, 64
    a, b = _inputs(M, N, K, 1, seed=3)
    ap = np.zeros((M, 72), np.uint16); ap[:, :K] = a[0]
    bp = np.zeros((N, 88), np.uint16); bp[:, :K] = b[0]
    p = G.run_gemm_softmax(ap, bp, M, N, K, alpha=0.125, lda=72, ldb=88, ldp=84)
    ref = oracle.gemm_softmax(oracle.widen(a, True), oracle.widen(b, True), M, N, K, alpha=0.125)
    P.assert_softmax_close(p.reshape(-1, N), ref.reshape(-1, N), tol=TOL)


def test_staged_write_out_widths_ragged_strips_and_leading_dimensions():
    # K = 64, N in {128, 256, 512}, fp32 P with 16-byte aligned rows: the 8-wave kernel whose probabilities leave
    # through LDS staging.  Ragged last strips (M not a multiple of 128), a batch that is not a multiple of 8,
    # several strips per workgroup with a shorter last group (17 strips x 64 matrices -> groups of 2), a padded
    # ldp that keeps the alignment (staged) and one that breaks it (the 4-wave kernel takes over).
    _check(200, 256, 64)
    _check(130, 128, 64, batch=3)
    _check(1000, 512, 64, batch=9, alpha=-0.25)
    _check(2100, 128, 64, batch=64)
    M, N, K = 150, 256, 64
    a, b = _inputs(M, N, K, 2, seed=5)
    ref = oracle.gemm_softmax(oracle.widen(a, True), oracle.widen(b, True), M, N, K, alpha=0.125, batch=2)
    for ldp in (260, 258):
        p = G.run_gemm_softmax(a, b, M, N, K, alpha=0.125, batch=2, ldp=ldp)
        P.assert_softmax_close(p.reshape(-1, N), ref.reshape(-1, N), tol=TOL)


@pytest.mark.parametrize("M,N,K,batch,ldp", [
    (1, 1, 8, 1, 1), (33, 3, 16, 2, 3), (31, 127, 24, 1, 127), (32, 128, 72, 3, 131), (65, 129, 64, 1, 129), (40, 255, 80, 2, 256),
    (33, 257, 136, 1, 257), (64, 512, 128, 2, 512), (17, 511, 200, 1, 511), (33, 513, 40, 32, 513), (1, 640, 64, 64, 640),
    (33, 641, 96, 32, 641), (20, 768, 80, 64, 768), (1, 769, 512, 64, 771), (33, 896, 64, 32, 896), (1, 897, 8, 65, 897),
    (33, 1023, 80, 32, 1023), (32, 1024, 64, 64, 1024), (70, 1020, 64, 64, 1021), (2, 1025, 64, 3, 1025),
    (33, 31, 40, 12, 31), (40, 63, 24, 9, 70), (32, 64, 128, 3, 64), (33, 65, 64, 10, 65),   # (2 waves up to 64 columns)
    (127, 128, 128, 2, 128), (128, 128, 128, 3, 128), (300, 128, 128, 9, 132),   # (127 rows here, 128 and more with B in the LDS)
])
def test_strip_kernel_edges(M, N, K, batch, ldp):
    # N at the edges of each column count per wave, K-steps that are partial, ragged strips, P of any alignment; the last
    # one is past the kernel's columns.  (Scaled by 1/sqrt(K): a score is a sum of K products of N(0,1) values, typically
    # off by sqrt(K) 2^-24 of its size sqrt(K), at most K 2^-24 sum |q||k|, and a probability by alpha times that: with
    # alpha = -0.5 at K = 512 fp32 accumulation alone costs 2e-5, 1.87e-5 was seen.)
    for alpha in (K ** -0.5, -2 * K ** -0.5):
        _check(M, N, K, alpha=alpha, batch=batch, ldp=ldp)
    _check(M, N, K, alpha=0.0, batch=batch, ldp=ldp)


@pytest.mark.parametrize("M,N,K,batch,ldp", [
    (33, 384, 72, 9, 384), (31, 385, 80, 9, 385), (17, 449, 128, 16, 452),      # three tiles per wave, then two with eight waves
    (33, 545, 96, 32, 545), (16, 673, 64, 64, 675), (32, 800, 128, 64, 800),    # three and four, whose last waves have none
    (32, 800, 136, 64, 800),                                                    # (two launches)
])
def test_strip_kernel_waves_and_tiles(M, N, K, batch, ldp):
    # both forms of the K-loop and of the write-out at the counts where they change, rows of 4 and 16 bytes' alignment
    test_strip_kernel_edges(M, N, K, batch, ldp)


@pytest.mark.parametrize("M,N,K,batch,ldp", [
    (16, 100, 64, 4, 100), (17, 100, 64, 4, 101), (49, 61, 72, 5, 61),    # stores from the registers from 17 rows of a strip on
    (33, 64, 64, 520, 64), (65, 127, 40, 200, 128),                       # ... and for no more of P than the caches hold
])
def test_strip_kernel_few_and_many(M, N, K, batch, ldp):
    test_strip_kernel_edges(M, N, K, batch, ldp)


@pytest.mark.parametrize("M,N,K", [(33, 5, 64), (40, 130, 128), (64, 512, 64), (1, 301, 128)])
def test_strip_kernel_bf16_output(M, N, K):
    _check(M, N, K, batch=3, p_bf16=True)


@pytest.mark.parametrize("M,N,K,batch", [(16, 100, 64, 4), (17, 103, 128, 4), (65, 127, 64, 200)])
def test_strip_kernel_bf16_output_few_and_many(M, N, K, batch):
    _check(M, N, K, batch=batch, p_bf16=True)


@pytest.mark.parametrize("M,N,K,batch,ldp", [
    (33, 383, 104, 257, 383), (1, 300, 264, 401, 300), (33, 509, 40, 257, 509),  # shared stages: three and four tiles
    (1, 514, 264, 769, 517), (33, 700, 24, 257, 700), (1, 768, 168, 769, 768),   # ... five and six
    (3, 577, 64, 257, 577), (17, 895, 104, 257, 896), (1, 1001, 168, 257, 1001),  # a wave's own: five, seven and eight
])
def test_strip_kernel_more_strips_than_the_chip_holds(M, N, K, batch, ldp):
    test_strip_kernel_edges(M, N, K, batch, ldp)


@pytest.mark.parametrize("M,N,K,batch", [(40, 384, 128, 3), (33, 381, 64, 257), (33, 385, 128, 3), (33, 499, 64, 257)])
def test_strip_kernel_bf16_output_tiles_and_waves(M, N, K, batch):
    _check(M, N, K, batch=batch, p_bf16=True)


def test_argmax_matches_scores():
    M, N, K = 256, 512, 64
    a, b = _inputs(M, N, K, 1, seed=7)
    p = G.run_gemm_softmax(a, b, M, N, K, alpha=0.125)[0]
    s = oracle.gemm(oracle.widen(a, True), oracle.widen(b, True), M, N, K, b_col=True, alpha=0.125)
    # the probabilities are monotone in the fp32 scores, which differ from the exact ones by
    # accumulation rounding: accept any column whose exact score is within that rounding of the best
    am = p.argmax(1)
    best = s.max(1)
    assert np.all(best - s[np.arange(M), am] <= 64 * 2.0 ** -24 * 64.0)


@pytest.mark.parametrize("M,N,K,batch", [(64, 1024, 64, 1), (100, 300, 256, 2), (33, 40, 48, 1), (70, 600, 64, 3)])
def test_two_operator_path(M, N, K, batch):
    # N > 512, K > 128 or K not a multiple of 32: scores through P, softmax in place
    _check(M, N, K, batch=batch)


def test_fp32_operands_take_the_two_operator_path():
    g = np.random.default_rng(2)
    M, N, K = 50, 60, 20
    a = g.standard_normal((M, K)).astype(np.float32)
    b = g.standard_normal((N, K)).astype(np.float32)
    p = G.run_gemm_softmax(a, b, M, N, K, alpha=0.3, ab_bf16=False)[0]
    ref = oracle.gemm_softmax(a.astype(np.float64), b.astype(np.float64), M, N, K, alpha=float(np.float32(0.3)))[0]
    P.assert_softmax_close(p, ref, tol=TOL)


def test_config4_full_size_sampled_batches_and_row_sums():
    import torch
    import paper_2511_03586_amd as perf
    wl = configs.CONFIG4
    d = wl.make()
    q, k = G.dev(d["q_bf16"].ravel()), G.dev(d["k_bf16"].ravel())
    S, D, B = wl.seq, wl.d, wl.batch
    p = torch.zeros(B * S * S, dtype=torch.float32, device="cuda")
    perf.perf_gemm_softmax(q.data_ptr(), k.data_ptr(), p.data_ptr(), S, S, D, D, D, S, B, S * D, S * D, S * S,
                           wl.alpha, perf.PERF_BF16, perf.PERF_F32, G.stream())
    torch.cuda.synchronize()
    sums = p.view(B * S, S).sum(1)
    assert float((sums - 1).abs().max()) <= 1e-5
    ph = p.view(B, S, S)
    for bi in (0, 1, 255, 511):
        ad, bd = oracle.widen(d["q_bf16"][bi], True), oracle.widen(d["k_bf16"][bi], True)
        ref = oracle.gemm_softmax(ad, bd, S, S, D, alpha=wl.alpha)[0]
        got = ph[bi].cpu().numpy()
        print(f"config 4 fused, matrix {bi}: max rel err {P.softmax_max_rel_err(got, ref)[0]:.3e}")
        P.assert_softmax_close(got, ref, tol=TOL)


def test_config4_full_size_every_entry_with_exact_scores():
    """Config 4's launch with small-integer operands (|q|, |k| <= 3): every product and partial sum
    is an integer below 2^24, so the fp32 scores are exact whatever the summation order, and
    alpha = 1/8 is a power of two. Every one of the 134M probabilities is then compared, at the
    1e-5 gate, with a float64 softmax of the exact integer scores computed on the host
    (numpy matmul), which is itself tied to the oracle on three matrices."""
    import torch
    import paper_2511_03586_amd as perf
    wl = configs.CONFIG4
    S, D, B = wl.seq, wl.d, wl.batch
    g = np.random.default_rng(404)
    qi = g.integers(-3, 4, (B, S, D)).astype(np.float32)
    ki = g.integers(-3, 4, (B, S, D)).astype(np.float32)
    q, k = G.dev(rng.f32_to_bf16_bits(qi).ravel()), G.dev(rng.f32_to_bf16_bits(ki).ravel())
    p = torch.zeros(B * S * S, dtype=torch.float32, device="cuda")
    perf.perf_gemm_softmax(q.data_ptr(), k.data_ptr(), p.data_ptr(), S, S, D, D, D, S, B, S * D, S * D, S * S,
                           wl.alpha, perf.PERF_BF16, perf.PERF_F32, G.stream())
    torch.cuda.synchronize()
    ph = p.view(B, S, S).cpu().numpy()
    worst = 0.0
    for b0 in range(0, B, 32):
        s = wl.alpha * np.matmul(qi[b0:b0 + 32].astype(np.float64), ki[b0:b0 + 32].astype(np.float64).transpose(0, 2, 1))
        e = np.exp(s - s.max(axis=-1, keepdims=True))
        ref = e / e.sum(axis=-1, keepdims=True)
        if b0 in (0, 256):
            bi = b0 + 5
            tie = oracle.gemm_softmax(qi[bi].astype(np.float64), ki[bi].astype(np.float64), S, S, D, alpha=wl.alpha)
            assert np.max(np.abs(tie.reshape(S, S) - ref[5]) / ref[5]) <= 1e-12
        rel, small = P.softmax_max_rel_err(ph[b0:b0 + 32].reshape(-1, S), ref.reshape(-1, S))
        worst = max(worst, rel)
        assert small <= 1e-35
    print(f"config 4 fused, exact scores, all {B * S * S} entries: max rel err {worst:.3e}")
    assert worst <= TOL


def test_deterministic():
    a, b = _inputs(256, 512, 64, 2, seed=9)
    p1 = G.run_gemm_softmax(a, b, 256, 512, 64, alpha=0.125, batch=2)
    p2 = G.run_gemm_softmax(a, b, 256, 512, 64, alpha=0.125, batch=2)
    assert np.array_equal(p1, p2)


def test_more_strips_than_a_launch_holds():
    """2^24 strips and more of 256 threads (a dimension of 2^32 threads is cut short without an error)."""
    import torch
    import paper_2511_03586_amd as perf
    batch, N, K = (1 << 24) + 3, 8, 8
    a = torch.ones((batch, K), dtype=torch.bfloat16, device="cuda")
    b = torch.zeros((N, K), dtype=torch.bfloat16, device="cuda")
    b[3] = 1.0
    p = torch.zeros((batch, N), dtype=torch.float32, device="cuda")
    perf.perf_gemm_softmax(a.data_ptr(), b.data_ptr(), p.data_ptr(), 1, N, K, K, K, N, batch, K, 0, N, 0.25, perf.PERF_BF16, perf.PERF_F32,
                           G.stream())
    want = torch.softmax(torch.tensor([0.0, 0, 0, 2, 0, 0, 0, 0], dtype=torch.float64), 0).to("cuda")
    assert bool(((p - want).abs() <= 1e-6).all())


@pytest.mark.parametrize("M,N,K", [(40, 60, 64), (40, 300, 128), (70, 500, 64), (300, 777, 80), (128, 512, 64)])
def test_nan_scores_are_not_probabilities(M, N, K):
    """A NaN among the operands makes NaN of the rows that it meets, in every kernel that keeps the scores in registers."""
    a, b = _inputs(M, N, K, 8)
    a[1, 5, 3] = 0x7FC0
    b[2, N - 1, 0] = 0xFFC1
    p = G.run_gemm_softmax(a, b, M, N, K, alpha=0.125, batch=8)
    assert np.all(np.isnan(p[1, 5])) and np.all(np.isnan(p[2]))
    p[1, 5], p[2] = 0, 0
    assert np.all(np.isfinite(p))
