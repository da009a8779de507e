"""Kernel variants: where a job's variants are different kernels each of them is run
against the oracle, and the autotuner compares them; where they are one kernel the
autotuner reports variant 0 with one time."""
import numpy as np
import pytest

import oracle
from paper_2302_05804_amd import synth
from tests.gpu_common import log, rel_l2, to_dev

pytestmark = pytest.mark.gpu


def _em():
    from paper_2302_05804_amd import em
    return em


def _context(prec, h, w, n, K, seed, x0):
    import torch
    em = _em()
    p = synth.make_problem("c2", H=h, W=w, n=n, K=K, seed=seed)
    x = torch.empty((h, w), dtype=torch.float32, device="cuda")
    ctx = em.Context(em.Problem.make(n, h, w, K, precision=getattr(em, prec)), to_dev(p.y), to_dev(p.v),
                     to_dev(p.psf), x, x0=to_dev(x0))
    return p, x, ctx


@pytest.mark.parametrize("prec,h,w,K", [
    ("BF16_SPLIT", 260, 300, 43), ("BF16_SPLIT", 140, 130, 25),   # 4 x 4 cells
    ("FP16_SPLIT", 96, 96, 43), ("FP16_SPLIT", 64, 200, 15),   # 64 x 64 tiles
])
def test_one_kernel_is_variant_0(prec, h, w, K):
    _, x, ctx = _context(prec, h, w, 3, K, 41, np.ones((h, w), np.float32))
    f, a, ms = ctx.autotune(2)
    log(f"{prec} {h}x{w} K={K}: {f}, {a}, {ms.tolist()}")
    ctx.close()
    assert (f, a) == (0, 0) and (ms > 0).all() and (ms == ms[:, :1]).all()


@pytest.mark.parametrize("prec,K", [("BF16_SPLIT", 15), ("BF16", 15), ("BF16", 43)])
def test_bf16_variants_match_oracle(prec, K):
    """Three layouts of the two-plane (K <= 15) and one-plane forms, in both directions."""
    h, w = 260, 300
    x0 = synth.positive_start((h, w), 5.0, seed=43)
    outs = []
    for fv in range(3):
        for av in range(3):
            p, x, ctx = _context(prec, h, w, 3, K, 42, x0)
            ctx.set_variants(fv, av)
            ctx.iterate(4)
            ctx.sync()
            outs.append(x.cpu().numpy())
            if fv == av == 0:
                _, _, ms = ctx.autotune(3)
                assert all(len(set(row)) == 3 for row in ms.tolist())
            ctx.close()
    xo = oracle.run(p.y, p.v, p.psf, x0, 4)
    errs = [rel_l2(o, xo) for o in outs]
    log(f"{prec} K={K}: rel L2 {min(errs):.2e} .. {max(errs):.2e}")
    # split form: 1e-4; plain BF16: 2^-9 per operand, four iterations
    assert max(errs) <= (1e-4 if prec == "BF16_SPLIT" else 4 * 2.0 ** -8)


def test_large_tile_fp16_variants_are_equal():
    """128 x 128 tiles in both directions (16 x 1024^2): the variants differ in their
    layout only, so their iterates are equal bit for bit."""
    h = w = 1024
    x0 = synth.positive_start((h, w), 20.0, seed=45)
    p, x, ctx = _context("FP16_SPLIT", h, w, 16, 43, 44, x0)
    _, _, ms = ctx.autotune(2)
    log(f"16 x 1024^2: {ms.tolist()}")
    assert all(len(set(row)) == 3 for row in ms.tolist())
    import torch
    outs = []
    for fv, av in ((0, 0), (1, 1), (2, 2), (0, 2), (2, 1)):
        x.copy_(to_dev(x0))
        torch.cuda.synchronize()
        ctx.set_variants(fv, av)
        ctx.iterate(3)
        ctx.sync()
        outs.append(x.cpu().numpy())
    ctx.close()
    assert all(np.array_equal(outs[0], o) for o in outs[1:])
