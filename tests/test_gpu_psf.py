"""GPU parity of the super-resolved PSF fit of Eq. (4) (em_psf_fit) against
the FP64 oracle (oracle.psf_fit), through the C ABI.

Both sides run the same projected-Adam iteration from the same start with the
same binary32 hyper-parameters; the GPU in binary32 (the blurred box-sum
factored as A h A^T), the oracle in binary64 from the definition.  Bar:
relative L2 of h <= 1e-4 and relative objective error <= 1e-4 (binary32 Adam
emulated on these problems stays within 4e-6 of binary64 after 2000 steps).
"""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2302_05804_amd import synth
from tests.gpu_common import log, rel_l2, to_dev

pytestmark = pytest.mark.gpu

H_BAR = 1e-4
OBJ_BAR = 1e-4


def _em():
    from paper_2302_05804_amd import em
    return em


def _oracle_kw(p):
    """The GPU problem's (binary32) hyper-parameters, for the oracle."""
    return dict(lam=float(p.lambda_), steps=int(p.n_steps), lr=float(p.lr), decay=float(p.lr_decay),
                beta1=float(p.beta1), beta2=float(p.beta2), eps=float(p.eps))


def _fit_both(f, kh, D, sigma, **kw):
    import torch
    em = _em()
    h, obj = em.psf_fit(to_dev(f), kh, D, sigma=sigma, **kw)
    torch.cuda.synchronize()
    p = em.psf_problem(f.shape[0], f.shape[1], kh, D, sigma=sigma, **kw)
    ho, oo = oracle.psf_fit(f, kh, D, sigma=float(p.sigma), **_oracle_kw(p))
    return h.cpu().numpy(), obj.cpu().numpy(), ho, oo


@pytest.mark.parametrize("n,kf,kh,D,sigma,lam,steps", [
    (3, 15, 15, 2, 2.0, 1e-2, 500),
    (2, 43, 43, 2, 2.0, 1e-2, 2000),     # the sizes of the super-resolution workload
    (2, 9, 21, 3, 3.0, 0.05, 300),
    (2, 7, 7, 1, 0.0, 0.5, 300),         # no blur, no down-sampling
    (1, 5, 63, 4, 0.7, 1e-3, 200),       # h wider than the fine stamp; largest h
    (1, 63, 63, 2, 2.0, 1e-2, 200),      # largest f and h
    (2, 1, 1, 1, 0.0, 0.0, 10),          # 1 x 1
    (1, 3, 5, 2, 1.0, 0.1, 100),
])
def test_fit_matches_oracle(n, kf, kh, D, sigma, lam, steps):
    log(f"psf fit n={n} Kf={kf} Kh={kh} D={D} sigma={sigma} lam={lam} steps={steps}")
    f = synth.coarse_psfs(n, kf, D, seed=kf * 31 + kh)
    hg, og, ho, oo = _fit_both(f, kh, D, sigma, lam=lam, steps=steps)
    err = rel_l2(hg, ho)
    oerr = float(np.abs(og - oo).max() / np.abs(oo).max()) if np.abs(oo).max() > 0 else 0.0
    log(f"  rel L2(h) {err:.2e}, objective rel err {oerr:.2e}, objective {oo.max():.3e}")
    assert (hg >= 0).all()
    assert err <= H_BAR and oerr <= OBJ_BAR


def test_constraint_binds():
    """f with negative lobes: the fit leaves pixels at exactly 0 on both sides."""
    rng = np.random.default_rng(61)
    f = synth.coarse_psfs(2, 15, 2, seed=62)
    f -= np.float32(0.3) * f.max() * (rng.uniform(size=f.shape) < 0.3).astype(np.float32)
    hg, og, ho, oo = _fit_both(f, 15, 2, 2.0, lam=1e-2, steps=800)
    zo = ho == 0
    log(f"  zeros: oracle {zo.sum()}, gpu {(hg == 0).sum()}; rel L2 {rel_l2(hg, ho):.2e}")
    assert zo.sum() > 0
    assert rel_l2(hg, ho) <= H_BAR


def test_zero_steps_and_explicit_start():
    import torch
    em = _em()
    f = synth.coarse_psfs(3, 11, 2, seed=63)
    f[0, 0, 0] = -0.01
    for D in (2, 4):
        h, obj = em.psf_fit(to_dev(f), 17, D, steps=0)
        torch.cuda.synchronize()
        ref = np.stack([oracle.psf_start(f[t], 17, D) for t in range(3)]).astype(np.float32)
        assert np.array_equal(h.cpu().numpy(), ref)
    h, _ = em.psf_fit(to_dev(f), 17, 3, steps=0)
    ref = np.stack([oracle.psf_start(f[t], 17, 3) for t in range(3)]).astype(np.float32)
    np.testing.assert_allclose(h.cpu().numpy(), ref, rtol=2 ** -23, atol=0)
    h0 = np.random.default_rng(64).uniform(0, 0.01, (3, 17, 17)).astype(np.float32)
    h, _ = em.psf_fit(to_dev(f), 17, 2, h0=to_dev(h0), steps=0)
    assert np.array_equal(h.cpu().numpy(), h0)
    hg, og = em.psf_fit(to_dev(f), 17, 2, h0=to_dev(h0), steps=150)
    p = em.psf_problem(3, 11, 17, 2, steps=150)
    ho, oo = oracle.psf_fit(f, 17, 2, h0=h0, sigma=float(p.sigma), **_oracle_kw(p))
    assert rel_l2(hg.cpu().numpy(), ho) <= H_BAR


def test_rejects_bad_arguments():
    import torch
    em = _em()
    f = to_dev(synth.coarse_psfs(2, 9, 2, seed=65))
    h = torch.empty((2, 9, 9), dtype=torch.float32, device="cuda")
    P = lambda t: ctypes.c_void_p(t.data_ptr())
    bad = [dict(psf_k=10), dict(out_k=65), dict(factor=5), dict(sigma=9.0), dict(lambda_=-1.0),
           dict(lr=-1.0), dict(lr_decay=0.0), dict(beta1=1.0), dict(eps=0.0), dict(n_steps=-1),
           dict(n_frames=0)]
    for b in bad:
        p = em.psf_problem(2, 9, 9, 2)
        for k, v in b.items():
            setattr(p, k, v)
        assert em._lib.em_psf_fit(ctypes.byref(p), P(f), None, P(h), None, None) == em.EINVAL, b
    p = em.psf_problem(2, 9, 9, 2, steps=5)
    assert em._lib.em_psf_fit(ctypes.byref(p), None, None, P(h), None, None) == em.EINVAL
    p = em.psf_problem(1 << 20, 9, 9, 2, steps=5)   # far more frames than the buffers hold
    assert em._lib.em_psf_fit(ctypes.byref(p), P(f), None, P(h), None, None) == em.EINVAL
    p = em.psf_problem(2, 9, 9, 2, steps=5)
    assert em._lib.em_psf_fit(ctypes.byref(p), P(f), None, P(h), None, None) == em.OK
    torch.cuda.synchronize()


def test_fitted_psfs_in_the_super_resolution_run():
    """Eq. (4) then Eq. (3): h fitted on each side from the same frame PSFs, then
    10 iterations of the sr = 2 update with those h (GPU FP32 vs oracle)."""
    import torch
    em = _em()
    n, hf, wf = 3, 40, 52
    f = synth.coarse_psfs(n, 43, 2, seed=66)
    hg, _ = em.psf_fit(to_dev(f), 43, 2, steps=1000)
    torch.cuda.synchronize()
    p = em.psf_problem(n, 43, 43, 2, steps=1000)
    ho, _ = oracle.psf_fit(f, 43, 2, sigma=float(p.sigma), **_oracle_kw(p))
    prob = synth.make_problem("c4", H=2 * hf, W=2 * wf, n=n, seed=67)
    x0 = synth.positive_start(prob.latent_shape, max(oracle.flat_x0(prob.y, prob.v, 2), 0.25), seed=68)
    from tests.gpu_common import gpu_run
    xg, _ = gpu_run(prob.y, prob.v, hg.cpu().numpy(), 2, 10, x0=x0)
    xo = oracle.run(prob.y, prob.v, ho.astype(np.float32), x0, 10, 2)
    err = rel_l2(xg, xo)
    log(f"  fitted-PSF SR run: rel L2(x) {err:.2e}")
    assert err <= 1e-4


def test_full_size_sampled_frames():
    """The workload the bench times (16 frame PSFs of 43 x 43, h 43 x 43,
    Delta = 2, 2000 steps) in one launch; two frames checked against the oracle."""
    import torch
    em = _em()
    f = synth.coarse_psfs(16, 43, 2, seed=4100)
    h, obj = em.psf_fit(to_dev(f), 43, 2)
    torch.cuda.synchronize()
    p = em.psf_problem(16, 43, 43, 2)
    for t in (0, 11):
        ho, oo = oracle.psf_fit(f[t:t + 1], 43, 2, sigma=float(p.sigma), **_oracle_kw(p))
        err = rel_l2(h[t].cpu().numpy(), ho[0])
        oerr = abs(float(obj[t]) - oo[0]) / oo[0]
        log(f"  frame {t}: rel L2(h) {err:.2e}, objective rel err {oerr:.2e}")
        assert err <= H_BAR and oerr <= OBJ_BAR


def test_paper_super_resolution_pipeline():
    """The super-resolution run as the paper describes it after Eq. (4): PSFs h
    fitted by Eq. (4) from the frame PSFs, exposures up-sampled to the fine grid,
    then the update of Eq. (2) on the fine grid with h.  Each side runs the whole
    pipeline itself (GPU: em_psf_fit, em_upsample, em_iterate; oracle: psf_fit,
    upsample, run); 8 iterations compared."""
    import torch
    em = _em()
    n, hf, wf = 3, 36, 44
    f = synth.coarse_psfs(n, 43, 2, seed=67)
    prob = synth.make_problem("c2", H=hf, W=wf, n=n, seed=68)     # frame-grid exposures
    hg, _ = em.psf_fit(to_dev(f), 43, 2, steps=1000)
    yu, vu = em.upsample(to_dev(prob.y), to_dev(prob.v), 2)
    torch.cuda.synchronize()
    p = em.psf_problem(n, 43, 43, 2, steps=1000)
    ho, _ = oracle.psf_fit(f, 43, 2, sigma=float(p.sigma), **_oracle_kw(p))
    yo, vo = oracle.upsample(prob.y, prob.v, 2)
    x0 = synth.positive_start((2 * hf, 2 * wf), max(oracle.flat_x0(yo, vo), 0.25), seed=69)
    from tests.gpu_common import gpu_run
    xg, _ = gpu_run(yu.cpu().numpy(), vu.cpu().numpy(), hg.cpu().numpy(), 1, 8, x0=x0)
    xo = oracle.run(yo, vo, ho.astype(np.float32), x0, 8, 1)
    err = rel_l2(xg, xo)
    log(f"  Eq. (4) + up-sampling + Eq. (2): rel L2(x) {err:.2e}")
    assert err <= 1e-4


@pytest.mark.parametrize("kf,kh", [(9, 15), (15, 43), (9, 63)])
@pytest.mark.parametrize("scale", [1e20, 1e30])
def test_overflowing_second_moments_stop_the_step(kf, kh, scale):
    """f finite but so large that Adam's second moments overflow: the step divides by
    an infinite root and is 0, so h keeps its start.  A step length of 0 keeps every
    other pixel too (0 times a finite quotient)."""
    import torch
    em = _em()
    f = (synth.coarse_psfs(2, kf, 2, seed=kf + kh).astype(np.float64) * scale).astype(np.float32)
    assert np.isfinite(f).all()
    h, _ = em.psf_fit(to_dev(f), kh, 2, lr=0.0, steps=5)
    torch.cuda.synchronize()
    start = np.stack([oracle.psf_start(f[t], kh, 2) for t in range(2)]).astype(np.float32)
    log(f"scale {scale:g} Kh={kh}: largest h {h.max():.3e}, start {start.max():.3e}")
    assert np.array_equal(h.cpu().numpy(), start)
