"""The 4 x 4 cell kernels (sr = 1, kernels padded to 43 x 43) at the edges of
their tiles, cells and 16-byte accesses, against the FP64 oracle.

FP32 runs on them from frames of 128 x 128 pixels on, as three bf16 parts per
operand: the split is exact, each product left out is below 2^-24 of the whole
one and at most three are, and a sum passes through fewer than 40 roundings of
2^-24, so every value is within (3 + 40) 2^-24 of the sum of the absolute
products.  BF16 split: 1e-4 of it, the bar of that form's operators.
"""
import numpy as np
import pytest

import oracle
from paper_2302_05804_amd import synth
from tests.gpu_common import gpu_run, log, rel_l2, to_dev

pytestmark = pytest.mark.gpu

FP32_BOUND = 43 * 2.0 ** -24
BF16_BOUND = 1e-4


def _em():
    from paper_2302_05804_amd import em
    return em


@pytest.mark.parametrize("hf,wf", [
    (128, 128),      # one BF16 tile, two FP32 tiles
    (129, 257),      # one row and one column into the next tiles
    (191, 130),      # odd height, width 2 mod 4
    (65, 515),       # width 3 mod 4
    (16385, 1), (8193, 2), (5462, 3), (4097, 5),   # narrower than one 16-byte access, or just wider
])
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_operators_at_tile_and_access_edges(prec, hf, wf):
    em = _em()
    code, bound = (em.FP32, FP32_BOUND) if prec == "fp32" else (em.BF16_SPLIT, BF16_BOUND)
    n, K = 2, 43
    rng = np.random.default_rng(hf * 1000 + wf)
    psf = rng.uniform(0, 1, (n, K, K)).astype(np.float32)
    psf /= psf.sum(axis=(1, 2), keepdims=True)
    # seven decades inside a tile
    x = np.exp(rng.uniform(np.log(1e-2), np.log(1e5), (hf, wf))).astype(np.float32)
    r = rng.normal(0, 1, (n, hf, wf)).astype(np.float32)
    p = em.Problem.make(n, hf, wf, K, precision=code)
    m = em.forward_op(p, to_dev(psf), to_dev(x)).cpu().numpy().astype(np.float64)
    s = em.adjoint_op(p, to_dev(psf), to_dev(r)).cpu().numpy().astype(np.float64)
    for t in range(n):
        mo, so = oracle.forward(psf[t], x, 1), oracle.adjoint(psf[t], r[t], 1)
        sa = oracle.adjoint(psf[t], np.abs(r[t]), 1)
        em_, es = np.abs(m[t] - mo) / mo, np.abs(s[t] - so) / sa
        log(f"{prec} {hf}x{wf} frame {t}: forward {em_.max():.2e}, adjoint {es.max():.2e} of the absolute sums")
        assert em_.max() <= bound and es.max() <= bound


@pytest.mark.parametrize("n", [1, 2, 5])
def test_fp32_frame_groups(n):
    """Frame counts that split unevenly over the groups of a small image."""
    p = synth.make_problem("c2", H=140, W=133, n=n, seed=310 + n)
    x0 = synth.positive_start(p.latent_shape, 20.0, seed=311)
    xg, trg = gpu_run(p.y, p.v, p.psf, 1, 4, x0=x0)
    xo, tro, _ = oracle.run(p.y, p.v, p.psf, x0, 4, trace=True)
    assert rel_l2(xg, xo) <= 1e-5
    assert np.abs(trg - tro).max() <= 1e-6 * np.abs(tro).max()


def test_fp32_large_and_small_values():
    """Near the largest binary32 the first part is clamped, not infinite."""
    em = _em()
    H, W, K = 130, 130, 43
    psf = np.zeros((1, K, K), np.float32)
    psf[0, 21, 21], psf[0, 0, 5] = 0.5, 0.25
    x = np.full((H, W), np.float32(3.4e38))
    x[:, 64:] = 1e-30
    p = em.Problem.make(1, H, W, K)
    m = em.forward_op(p, to_dev(psf), to_dev(x)).cpu().numpy()[0].astype(np.float64)
    mo = oracle.forward(psf[0], x, 1)
    assert np.isfinite(m).all()
    assert np.abs(m / mo - 1).max() <= FP32_BOUND


@pytest.mark.parametrize("hf,wf,n", [
    (64, 64, 4),       # one adjoint tile down, whole four-frame products
    (65, 131, 5),      # one row and column into the next tiles, three frames of a product empty
    (33, 130, 1), (8192, 1, 2), (2100, 2, 3),
])
def test_fp32_sr2_operators_at_tile_edges(hf, wf, n):
    em = _em()
    K = 43
    rng = np.random.default_rng(hf * 7 + wf)
    psf = rng.uniform(0, 1, (n, K, K)).astype(np.float32)
    psf /= psf.sum(axis=(1, 2), keepdims=True)
    x = np.exp(rng.uniform(np.log(1e-2), np.log(1e5), (2 * hf, 2 * wf))).astype(np.float32)
    r = rng.normal(0, 1, (n, hf, wf)).astype(np.float32)
    p = em.Problem.make(n, hf, wf, K, sr=2)
    m = em.forward_op(p, to_dev(psf), to_dev(x)).cpu().numpy().astype(np.float64)
    s = em.adjoint_op(p, to_dev(psf), to_dev(r)).cpu().numpy().astype(np.float64)
    # one more rounding: the taps of the box-extended kernel
    bound = FP32_BOUND + 2.0 ** -24
    for t in range(n):
        mo, so = oracle.forward(psf[t], x, 2), oracle.adjoint(psf[t], r[t], 2)
        sa = oracle.adjoint(psf[t], np.abs(r[t]), 2)
        ef, ea = np.abs(m[t] - mo) / mo, np.abs(s[t] - so) / sa
        log(f"sr=2 {hf}x{wf} frame {t}: forward {ef.max():.2e}, adjoint {ea.max():.2e} of the absolute sums")
        assert ef.max() <= bound and ea.max() <= bound


@pytest.mark.parametrize("sr", [1, 2])
def test_fp32_single_products(sr):
    """One tap: every output is one product (sr = 2: of the adjoint).  FP32 holds it to
    half a unit, 2^-24; here the sum of the largest part product with the seven
    others (below 2^-7 of it, seven roundings of 2^-24) rounds once more, and the
    ninth is below 2^-32: 2^-24 (1 + 2^-3) in all."""
    em = _em()
    n, H, W, K = 2, 130 // sr, 260 // sr, 43
    rng = np.random.default_rng(905 + sr)
    psf = np.zeros((n, K, K), np.float32)
    psf[0, 21, 21], psf[1, 3, 40] = rng.uniform(0.1, 1, 2)
    bound = 2.0 ** -24 * (1 + 2.0 ** -3)
    p = em.Problem.make(n, H, W, K, sr=sr)
    r = np.exp(rng.uniform(-5, 5, (n, H, W))).astype(np.float32)
    s = em.adjoint_op(p, to_dev(psf), to_dev(r)).cpu().numpy().astype(np.float64)
    pairs = [(s[t], oracle.adjoint(psf[t], r[t], sr)) for t in range(n)]
    if sr == 1:
        x = np.exp(rng.uniform(-5, 5, (H, W))).astype(np.float32)
        m = em.forward_op(p, to_dev(psf), to_dev(x)).cpu().numpy().astype(np.float64)
        pairs += [(m[t], oracle.forward(psf[t], x, 1)) for t in range(n)]
    for got, want in pairs:
        at = want > 0
        err = np.abs(got[at] / want[at] - 1).max()
        log(f"sr={sr} one tap: largest error {err / 2.0 ** -24:.4f} x 2^-24")
        assert (got[~at] == 0).all() and err <= bound


@pytest.mark.parametrize("sr,hf,wf,n,groups", [
    (1, 1024, 1024, 8, 2), (1, 940, 2100, 15, 1), (2, 471, 1050, 15, 1), (2, 200, 300, 33, 7),
])
def test_fp32_frame_sums(sr, hf, wf, n, groups):
    """The sum over frames is held in FP64: one tap of 1, unit weights, so that B is
    the plain sum of the exposures.  The frame groups' sums are rounded once (2^-24 of
    the total together) and added in FP32 (2^-24 for each further group).  A chain over
    15 frames in FP32 is off by up to 15 times that."""
    import torch
    em = _em()
    g = torch.Generator(device="cuda").manual_seed(hf + n)
    y = torch.rand((n, hf, wf), generator=g, device="cuda") + 0.5
    v = torch.ones_like(y)
    psf = torch.zeros((n, 43, 43), device="cuda")
    psf[:, 21, 21] = 1.0
    p = em.Problem.make(n, hf, wf, 43, sr=sr)
    x = torch.empty(p.latent_shape, device="cuda")
    ctx = em.Context(p, y, v, psf, x)
    B, _ = ctx.terms()
    ctx.sync()
    want = y.double().sum(0)
    if sr == 2:
        want = want.repeat_interleave(2, 0).repeat_interleave(2, 1)
    err = float((B.double() / want - 1).abs().max()) / 2.0 ** -24
    log(f"sr={sr} {n} x {hf} x {wf}: largest error of the frame sum {err:.3f} x 2^-24")
    ctx.close()
    assert err <= groups + 0.01


@pytest.mark.parametrize("sr", [1, 2])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_fp32_operators_with_non_finite_pixels(sr, bad):
    """Pixels that are infinite or NaN reach the outputs of their 43 x 43 support (44 x
    44 latent pixels for sr = 2) and no others.  All taps are positive, so an infinity
    gives infinities, as a plain sum does."""
    em = _em()
    n, H, W, K = 3, 270 // sr, 390 // sr, 43
    rng = np.random.default_rng(77)
    psf = rng.uniform(0.1, 1, (n, K, K)).astype(np.float32)
    psf /= psf.sum(axis=(1, 2), keepdims=True)
    x = rng.uniform(1, 2, (sr * H, sr * W)).astype(np.float32)
    r = rng.uniform(-1, 1, (n, H, W)).astype(np.float32)
    x[0, 7] = x[131, 258] = bad
    r[1, 60, 90] = r[2, 0, W - 1] = bad
    p = em.Problem.make(n, H, W, K, sr=sr)
    m = em.forward_op(p, to_dev(psf), to_dev(x)).cpu().numpy().astype(np.float64)
    s = em.adjoint_op(p, to_dev(psf), to_dev(r)).cpu().numpy().astype(np.float64)
    for t in range(n):
        xa, ra = np.nan_to_num(np.abs(x), posinf=0), np.nan_to_num(np.abs(r[t]), posinf=0)
        for got, want, absum in ((m[t], oracle.forward(psf[t], x, sr), oracle.forward(psf[t], xa, sr)),
                                 (s[t], oracle.adjoint(psf[t], r[t], sr), oracle.adjoint(psf[t], ra, sr))):
            fin = np.isfinite(want)
            assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[~fin], want[~fin], equal_nan=True)
            assert (np.abs(got[fin] - want[fin]) <= (FP32_BOUND + 2.0 ** -24) * absum[fin]).all()


@pytest.mark.parametrize("sr", [1, 2])
@pytest.mark.parametrize("xs,fs", [(1e-37, 1.0), (1e-41, 1.0), (1e4, 1e-37), (1e25, 1e-38), (1e-20, 1e-14),
                                   (2e18, 1.0), (1e36, 1e-1)])
def test_fp32_tiny_and_huge_operands(sr, xs, fs):
    """Operands down to the subnormal numbers are held exactly: the error is that of
    the sum (FP32_BOUND of the absolute sum; one tap more for the box) and of rounding
    the result, half of 2^-149 at least."""
    em = _em()
    n, H, W, K = 2, 132 // sr, 260 // sr, 43
    rng = np.random.default_rng(31)
    psf = rng.uniform(0, 1, (n, K, K))
    psf = (psf / psf.sum(axis=(1, 2), keepdims=True) * 40 * fs).astype(np.float32)
    x = (rng.uniform(0.5, 1, (sr * H, sr * W)) * xs).astype(np.float32)
    r = (rng.uniform(0.5, 1, (n, H, W)) * xs).astype(np.float32)
    if fs < 1e-30:
        psf[1] = 0
        psf[1, 5, 30] = 3.3 * fs
    p = em.Problem.make(n, H, W, K, sr=sr)
    m = em.forward_op(p, to_dev(psf), to_dev(x)).cpu().numpy().astype(np.float64)
    s = em.adjoint_op(p, to_dev(psf), to_dev(r)).cpu().numpy().astype(np.float64)
    for t in range(n):
        for got, want in ((m[t], oracle.forward(psf[t], x, sr)), (s[t], oracle.adjoint(psf[t], r[t], sr))):
            err = np.abs(got - want)
            # a box tap is rounded to binary32, where the smallest step is 2^-149
            tap = 0.5 * 2.0 ** -149 * x.sum(dtype=np.float64) if sr == 2 else 0.0
            assert (err <= (FP32_BOUND + 2.0 ** -24) * want + 2.0 ** -150 * 1.001 + tap).all()
