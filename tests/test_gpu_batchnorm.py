"""GPU parity: perf_batchnorm against the CPU oracle. Tolerances as for LayerNorm: mean, rstd and
fp32 outputs 1e-5 relative (output denominator floored at the channel's RMS, mean's at 1e-3),
bf16 outputs within one bf16 ulp of the oracle's single rounding."""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_03586_amd as perf
from workloads import rng
from tests import gpu_helpers as G
from tests import parity as P

pytestmark = pytest.mark.gpu


def _run(x, gamma, beta, eps, x_bf16, p_bf16, y_bf16, inplace=False, want_stats=True):
    N, C, H, W = x.shape
    xd, gd, bd = G.dev(x.ravel()), G.dev(gamma), G.dev(beta)
    yd = xd if inplace else torch.zeros(x.size, dtype=torch.int16 if y_bf16 else torch.float32, device="cuda")
    md = torch.zeros(C, dtype=torch.float32, device="cuda")
    rd = torch.zeros(C, dtype=torch.float32, device="cuda")
    nbytes = perf.perf_batchnorm_workspace_bytes(N, C, H, W)
    assert nbytes > 0
    ws = torch.full((nbytes // 4 + 8,), float("nan"), dtype=torch.float32, device="cuda")   # scratch starts as garbage
    perf.perf_batchnorm(xd.data_ptr(), gd.data_ptr(), bd.data_ptr(), yd.data_ptr(), md.data_ptr() if want_stats else None,
                        rd.data_ptr() if want_stats else None, ws.data_ptr(), N, C, H, W, eps, G.dt(x_bf16), G.dt(p_bf16),
                        G.dt(y_bf16), G.stream())
    torch.cuda.synchronize()
    assert bool(torch.isnan(ws[nbytes // 4:]).all()), "kernel wrote past the workspace it asked for"
    return G.host(yd, y_bf16).reshape(x.shape), md.cpu().numpy(), rd.cpu().numpy()


def _check(N, C, H, W, x_bf16=False, p_bf16=False, y_bf16=False, seed=0, offsets=None, **kw):
    g = np.random.default_rng(seed)
    sig = g.uniform(0.5, 3.0, C)
    off = np.asarray(offsets if offsets is not None else g.uniform(-3, 3, C))
    x = (g.standard_normal((N, C, H, W)) * sig[None, :, None, None] + off[None, :, None, None]).astype(np.float32)
    gamma = g.uniform(0.5, 1.5, C).astype(np.float32)
    beta = (g.standard_normal(C) * 0.3).astype(np.float32)
    xs = rng.f32_to_bf16_bits(x) if x_bf16 else x
    gs, bs = (rng.f32_to_bf16_bits(gamma), rng.f32_to_bf16_bits(beta)) if p_bf16 else (gamma, beta)
    y, m, r = _run(xs, gs, bs, 1e-5, x_bf16, p_bf16, y_bf16, **kw)
    ref, mref, rref = oracle.batchnorm(oracle.widen(xs, x_bf16), oracle.widen(gs, p_bf16), oracle.widen(bs, p_bf16),
                                       float(np.float32(1e-5)))
    if kw.get("want_stats", True):
        assert np.max(np.abs(m - mref) / np.maximum(np.abs(mref), 1e-3)) <= 1e-5
        assert np.max(np.abs(r - rref) / rref) <= 1e-5
    if y_bf16:
        got, want = P.bf16_to_f64(y), P.bf16_to_f64(oracle.round_bf16(ref))
        assert np.all(np.abs(got - want) <= 2.0 ** -7 * np.maximum(np.abs(ref), 2.0 ** -7))
        # bf16 inputs repeat values, and a channel shares one (mean, scale): when an input value maps
        # next to a rounding tie every occurrence flips together, so the identical fraction is
        # gated loosely here (measured 99.8 % on the smallest case, statistics exact to 5e-8)
        assert np.mean(got == want) >= 0.99
    else:
        rms = np.sqrt(np.mean(ref ** 2, axis=(0, 2, 3), keepdims=True))
        assert np.max(np.abs(y - ref) / np.maximum(np.abs(ref), rms)) <= 1e-5


@pytest.mark.parametrize("N,C,H,W", [(8, 64, 300, 300), (2, 3, 512, 512), (1, 1, 1, 1), (3, 5, 7, 9), (2, 4, 129, 127),
                                     (4, 2, 128, 130), (1, 7, 1, 40000), (16, 16, 8, 8)])
def test_shapes_fp32(N, C, H, W):
    _check(N, C, H, W)


def test_dtypes_inplace_and_no_stats():
    _check(4, 8, 64, 66, x_bf16=True, y_bf16=True)
    _check(4, 8, 64, 66, x_bf16=True, p_bf16=True, y_bf16=False)
    _check(2, 6, 40, 40, x_bf16=False, y_bf16=True)
    _check(2, 6, 33, 35, x_bf16=True, y_bf16=True)          # odd plane size: element path
    _check(3, 4, 50, 52, inplace=True)
    _check(3, 4, 50, 52, want_stats=False)


def test_large_offset_channels_and_constant_channel():
    # mean >> sigma: the shifted-moment partials and the double-precision merge keep 1e-5
    _check(4, 3, 200, 200, offsets=[1e3, -2e3, 0.0], seed=5)
    x = np.empty((2, 2, 16, 16), np.float32); x[:, 0] = 7.0
    x[:, 1] = (2.0 * (-1.0) ** np.arange(16))[None, None, :]
    y, m, r = _run(x, np.array([1.5, 1.5], np.float32), np.array([0.25, -1.0], np.float32), 1e-5, False, False, False)
    assert np.all(y[:, 0] == 0.25) and m[0] == 7.0
    np.testing.assert_allclose(y[:, 1], x[:, 1] / np.sqrt(4.0 + 1e-5) * 1.5 - 1.0, rtol=2e-6)


def test_deterministic():
    g = np.random.default_rng(1)
    x = g.standard_normal((4, 6, 100, 100)).astype(np.float32)
    a = _run(x, np.ones(6, np.float32), np.zeros(6, np.float32), 1e-5, False, False, False)
    b = _run(x, np.ones(6, np.float32), np.zeros(6, np.float32), 1e-5, False, False, False)
    assert all(np.array_equal(u, v) for u, v in zip(a, b))


@pytest.mark.parametrize("N,C,H,W", [
    (5, 3, 1, 3), (9, 4, 1, 5),              # planes shorter than 16 bytes (both types, bf16 only)
    (7, 700, 5, 7), (40, 30, 13, 13),        # planes grouped to a segment, a shorter last group, odd planes
    (6, 512, 16, 16), (3, 4, 90, 91),        # ... whole aligned chunks; one plane to a segment
    (3, 4, 1, 8193), (2, 3, 1, 16387), (2, 2, 1, 49152),   # split planes: a ragged last segment, one of 3 elements, whole ones
    (4096, 1, 2, 1), (2731, 3, 1, 3),        # many short planes: 256 and 1024 threads
    (1, 2, 2100, 2000),                      # more than 256 segments per channel: merged by a kernel of their own
])
def test_segment_edges(N, C, H, W):
    _check(N, C, H, W, inplace=True)
    _check(N, C, H, W, x_bf16=True, y_bf16=True, inplace=True)
    _check(N, C, H, W, x_bf16=True, p_bf16=True)
    _check(N, C, H, W, y_bf16=True)


@pytest.mark.parametrize("x_bf16,y_bf16", [(False, False), (True, True), (True, False)])
@pytest.mark.parametrize("N,C,H,W", [
    (1, 3, 2, 4), (2, 2, 16, 32), (3, 2, 3, 3), (4, 3, 11, 23),      # 256 threads: one chunk in all, every thread's full, ragged planes
    (8, 2, 8, 64), (5, 2, 25, 33), (16, 2, 32, 32), (4, 2, 65, 63),  # 1024 threads, full and ragged; as many chunks as are held
    (1, 1, 129, 128), (1, 1, 127, 257),                              # one row more than that (fp32): two launches
])
def test_channels_in_one_workgroup(N, C, H, W, x_bf16, y_bf16):
    _check(N, C, H, W, x_bf16=x_bf16, y_bf16=y_bf16, seed=N + W)
    # (the mean is an fp32 number: half a unit in its last place, 2^-20 at 30, over a deviation of 0.2 and more is under 1e-5)
    _check(N, C, H, W, x_bf16=x_bf16, y_bf16=y_bf16, seed=N + W, offsets=[30.0] * C, inplace=x_bf16 == y_bf16, want_stats=False)


@pytest.mark.parametrize("y_bf16", [True, False])
@pytest.mark.parametrize("N,C,H,W", [
    (16, 2, 40, 44), (16, 2, 112, 18),             # whole chunks, the most in one launch and more
    (16, 2, 31, 33), (17, 2, 31, 33),              # ragged ones
    (32, 16, 7, 127), (32, 17, 7, 127),            # the most planes that are spread
    (14, 2, 32, 64), (13, 2, 33, 72), (4, 2, 63, 71), (4, 2, 63, 73),   # the longest, whole and ragged
])
def test_bf16_channels_in_one_launch_or_two(N, C, H, W, y_bf16):
    _check(N, C, H, W, x_bf16=True, y_bf16=y_bf16, seed=N + W, inplace=y_bf16)


@pytest.mark.parametrize("ratio", [1e4, 1e5, 1e6, 3e6])
@pytest.mark.parametrize("N,C,H,W", [(2, 16, 16, 32), (4, 16, 31, 33), (4, 16, 64, 64)])   # 256 and 1024 threads, whole and ragged
def test_one_workgroup_large_offsets(N, C, H, W, ratio):
    """Means of up to 3e6 deviations, and a constant channel whose value 16 bits do not hold. An element's square meets at most
    4 roundings in its chunk, 4 over the thread's chunks and 6 in the wave; the moment about the provisional mean is at
    most 5/4 of the one about the mean: the variance is within 1.25 * 14 * 2^-24, its root within half of that."""
    g = np.random.default_rng(int(ratio) + H)
    x = (g.standard_normal((N, C, H, W)) + ratio * (1 + np.arange(C) / C)[None, :, None, None]).astype(np.float32)
    x[:, 0] = np.float32(ratio * 1.2345678)
    gamma, beta, eps = g.uniform(0.5, 1.5, C).astype(np.float32), np.zeros(C, np.float32), float(np.float32(1e-5))
    y, m, r = _run(x, gamma, beta, eps, False, False, False)
    x = x.astype(np.float64)
    mean = x.mean(axis=(0, 2, 3))
    rstd = 1 / np.sqrt(np.square(x - mean[None, :, None, None]).mean(axis=(0, 2, 3)) + eps)
    assert np.max(np.abs(m - mean) / mean) <= 2.0 ** -23
    assert np.max(np.abs(r - rstd) / rstd) <= 0.625 * 14 * 2.0 ** -24 + 2.0 ** -24
    want = (x - m.astype(np.float64)[None, :, None, None]) * (rstd * gamma)[None, :, None, None]
    assert np.all(np.abs(y - want) <= 1e-6 * np.abs(want) + 1e-6)


def test_one_workgroup_nan_stays_in_its_channel():
    x = np.random.default_rng(0).standard_normal((2, 3, 8, 9)).astype(np.float32)
    x[1, 1, 3, 3] = np.nan
    y, m, r = _run(x, np.ones(3, np.float32), np.zeros(3, np.float32), 1e-5, False, False, False)
    assert np.isnan(y[:, 1]).all() and np.isnan(m[1]) and np.isnan(r[1])
    assert np.isfinite(y[:, [0, 2]]).all() and np.isfinite(m[[0, 2]]).all()
