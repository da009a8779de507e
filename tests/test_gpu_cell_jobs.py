"""Whole jobs and operators on the 4 x 4 cell kernels where their epilogues, their
zero-padded kernels and their unaligned accesses can go wrong: Student-t noise with
the log-likelihood traced, kernel sides between 17 and 41, buffers that are only
4-byte aligned, and the job that em_run_noalloc takes on its smallest plan.
FP32 takes these kernels from 16384 latent pixels on.
Bars: x rel L2 <= 1e-5 and log-likelihood 1e-6 (FP32), 1e-3 (BF16 split); operators
as in test_gpu_cell.py."""
import numpy as np
import pytest

import oracle
from paper_2302_05804_amd import synth
from tests.gpu_common import log, rel_l2, to_dev

pytestmark = pytest.mark.gpu

# 43 roundings of 2^-24 of the absolute sum, one more for the taps of the box-extended kernel
FP32_BOUND = 44 * 2.0 ** -24
BF16_BOUND = 1e-4
# plain BF16: 2^-9 for each operand
PLAIN_BOUND = 2.0 ** -8


def _em():
    from paper_2302_05804_amd import em
    return em


@pytest.mark.parametrize("sr,hf,wf,n,K", [
    (1, 131, 133, 3, 43),     # odd width
    (1, 130, 258, 2, 43),     # width 2 mod 4
    (1, 128, 132, 4, 31),     # width a multiple of 4
    (2, 131, 67, 5, 43),      # odd width, three of eight frame slots empty
    (2, 66, 70, 6, 43),       # even width
    (2, 64, 64, 4, 25),       # whole products and tiles
])
def test_student_t_runs(sr, hf, wf, n, K):
    import torch
    em = _em()
    p = synth.make_problem("c4" if sr == 2 else "c2", H=sr * hf, W=sr * wf, n=n, K=K, seed=8100 + wf)
    y, hit = synth.add_trails(p.y, p.v, 8200 + wf)
    nu, it = 3.0, 4
    x0 = synth.positive_start(p.latent_shape, max(oracle.flat_x0(y, p.v, sr), 0.25), seed=8300)
    prob = em.Problem.make(n, hf, wf, K, sr=sr, nu=nu)
    assert hit.any() and prob.latent_shape[0] * prob.latent_shape[1] >= 16384
    x = torch.empty(prob.latent_shape, dtype=torch.float32, device="cuda")
    ctx = em.Context(prob, to_dev(y), to_dev(p.v), to_dev(p.psf), x, x0=to_dev(x0))
    B, Dn = ctx.terms()
    tr = ctx.iterate(it, trace=True)
    ll = ctx.loglik()
    ctx.close()
    Bo, Do = oracle.terms_t(y, p.v, p.psf, x0, nu, sr)
    xo, tro, _ = oracle.run_t(y, p.v, p.psf, x0, it, nu, sr, trace=True)
    err, llerr = rel_l2(x.cpu().numpy(), xo), float(np.abs(tr - tro).max() / np.abs(tro).max())
    eb, ed = rel_l2(B.cpu().numpy(), Bo), rel_l2(Dn.cpu().numpy(), Do)
    log(f"Student-t sr={sr} {n} x {hf} x {wf} K={K}: x {err:.2e}, loglik {llerr:.2e}, B {eb:.2e}, Dn {ed:.2e}")
    assert err <= 1e-5 and llerr <= 1e-6 and eb <= 1e-5 and ed <= 1e-5
    assert abs(ll - oracle.loglik_t(y, p.v, p.psf, xo, nu, sr)) <= 1e-6 * abs(ll)


@pytest.mark.parametrize("K", [17, 25, 31, 41])
@pytest.mark.parametrize("prec,sr", [("FP32", 1), ("FP32", 2), ("BF16_SPLIT", 1), ("BF16", 1)])
def test_operators_of_padded_kernels(prec, sr, K):
    em = _em()
    bound = {"FP32": FP32_BOUND, "BF16_SPLIT": BF16_BOUND, "BF16": PLAIN_BOUND}[prec]
    n, hf, wf = 3, 134 // sr, 150 // sr
    rng = np.random.default_rng(K * 10 + sr)
    psf = rng.uniform(0, 1, (n, K, K)).astype(np.float32)
    psf /= psf.sum(axis=(1, 2), keepdims=True)
    x = np.exp(rng.uniform(-4, 8, (sr * hf, sr * wf))).astype(np.float32)
    r = rng.normal(0, 1, (n, hf, wf)).astype(np.float32)
    p = em.Problem.make(n, hf, wf, K, sr=sr, precision=getattr(em, prec))
    m = em.forward_op(p, to_dev(psf), to_dev(x)).cpu().numpy().astype(np.float64)
    s = em.adjoint_op(p, to_dev(psf), to_dev(r)).cpu().numpy().astype(np.float64)
    for t in range(n):
        mo, so = oracle.forward(psf[t], x, sr), oracle.adjoint(psf[t], r[t], sr)
        sa = oracle.adjoint(psf[t], np.abs(r[t]), sr)
        ef, ea = (np.abs(m[t] - mo) / mo).max(), (np.abs(s[t] - so) / sa).max()
        log(f"{prec} sr={sr} K={K} frame {t}: forward {ef:.2e}, adjoint {ea:.2e}")
        assert ef <= bound and ea <= bound


@pytest.mark.parametrize("prec,sr,nu", [("FP32", 1, 0.0), ("FP32", 1, 3.0), ("FP32", 2, 0.0), ("FP32", 2, 3.0),
                                        ("BF16_SPLIT", 1, 0.0)])
def test_buffers_on_4_byte_boundaries(prec, sr, nu):
    """Widths that are a multiple of 4 with buffers that are not 16-byte aligned: the
    accesses change, the values do not."""
    import torch
    em = _em()
    n, hf, wf, K = 3, 136 // sr, 144 // sr, 43
    p = synth.make_problem("c4" if sr == 2 else "c2", H=sr * hf, W=sr * wf, n=n, K=K, seed=8400)
    prob = em.Problem.make(n, hf, wf, K, sr=sr, precision=getattr(em, prec), nu=nu)
    outs = []
    for shift in (0, 1, 3):
        def buf(a):
            t = to_dev(a)
            b = torch.empty(t.numel() + 4, device="cuda")[shift:shift + t.numel()].view(t.shape)
            b.copy_(t)
            return b
        x0 = buf(synth.positive_start(p.latent_shape, 5.0, seed=8401))
        x = buf(np.zeros(p.latent_shape, np.float32))
        ctx = em.Context(prob, buf(p.y), buf(p.v), buf(p.psf), x, x0=x0)
        tr = ctx.iterate(3, trace=True)
        ctx.sync()
        ctx.close()
        m, s = buf(np.zeros(p.y.shape, np.float32)), buf(np.zeros((n,) + tuple(p.latent_shape), np.float32))
        em.forward_op(prob, buf(p.psf), x0, m=m)
        em.adjoint_op(prob, buf(p.psf), buf(np.nan_to_num(p.y)), s=s)
        torch.cuda.synchronize()
        outs.append([tr] + [t.cpu().numpy() for t in (x, m, s)])
    for o in outs[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(outs[0], o))


def test_noalloc_on_the_smallest_plan():
    """33 x 964^2 in FP32: with the matrix-core tables the workspace is beyond the
    static scratch, without them it fits, and the call runs the direct convolution.
    Both are FP32: the iterates agree to 1e-6."""
    import torch
    em = _em()
    n, h, w, K = 33, 964, 964, 43
    prob = em.Problem.make(n, h, w, K)
    assert em.workspace_bytes(prob) > em.NOALLOC_SCRATCH_BYTES
    g = torch.Generator(device="cuda").manual_seed(9)
    y = torch.rand((n, h, w), generator=g, device="cuda") * 50 + 5
    v = torch.rand((n, h, w), generator=g, device="cuda") * 9 + 1
    f = torch.rand((n, K, K), generator=g, device="cuda")
    f /= f.sum(dim=(1, 2), keepdim=True)
    x0 = torch.rand((h, w), generator=g, device="cuda") * 20 + 1
    a, b = torch.empty((h, w), device="cuda"), torch.empty((h, w), device="cuda")
    ta = em.run_noalloc(prob, y, v, f, a, 2, x0=x0, trace=True)
    ctx = em.Context(prob, y, v, f, b, x0=x0)
    tb = ctx.iterate(2, trace=True)
    ctx.close()
    err = float((a.double() - b.double()).norm() / b.double().norm())
    log(f"smallest plan: rel L2 {err:.2e}, loglik {np.abs(ta / tb - 1).max():.2e}")
    assert err <= 1e-6 and np.abs(ta / tb - 1).max() <= 1e-7


@pytest.mark.parametrize("nu", [0.0, 3.0])
def test_served_plain_bf16(nu):
    """Served plain BF16 jobs run on the cells (alone they do not): two jobs of ragged
    sizes in one round, each against the oracle (2^-9 for each operand, four iterations)."""
    em = _em()
    srv = em.Server(256 << 20, max_slots=2)
    jobs = []
    for k, (h, w, n, K) in enumerate([(131, 205, 3, 43), (96, 77, 5, 31)]):
        p = synth.make_problem("c2", H=h, W=w, n=n, K=K, seed=8600 + k)
        y = synth.add_trails(p.y, p.v, 8700 + k)[0] if nu else p.y
        jid = srv.submit(em.Problem.make(n, h, w, K, precision=em.BF16, nu=nu), y, p.v, p.psf, 4)
        jobs.append((p, y, jid))
    for p, y, jid in jobs:
        x, ll = srv.wait(jid)
        x0 = np.full(p.latent_shape, oracle.flat_x0(y, p.v), np.float32)
        xo = oracle.run_t(y, p.v, p.psf, x0, 4, nu) if nu else oracle.run(y, p.v, p.psf, x0, 4)
        lo = oracle.loglik_t(y, p.v, p.psf, xo, nu) if nu else oracle.loglik(y, p.v, p.psf, xo)
        err = rel_l2(x, xo)
        log(f"served BF16 nu={nu} {y.shape}: x {err:.2e}, loglik {abs(ll / lo - 1):.2e}")
        assert err <= 4 * 2.0 ** -8 and abs(ll / lo - 1) <= 4 * 2.0 ** -8
    srv.close()
