"""Small images take smaller tiles (FP16 split, sr = 1: 64 x 64 instead of 128 x 128
outputs per workgroup; FP32 direct convolution: 16 instead of 64 rows).  A tile's
shape does not enter the sums, so a job run alone on small tiles equals, bit for
bit, the same job served, which always takes the large ones (and never splits the
frame sum: the sizes here have one frame to a group)."""
import numpy as np
import pytest

from paper_2302_05804_amd import synth
from tests.gpu_common import gpu_run, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,K,h,w,n", [
    ("FP16_SPLIT", 43, 64, 64, 3), ("FP16_SPLIT", 43, 65, 130, 2), ("FP16_SPLIT", 15, 129, 63, 4),
    ("FP16_SPLIT", 31, 500, 500, 8),
    ("FP16_SPLIT", 15, 65, 769, 40),     # small tiles in the adjoint only
    ("FP16_SPLIT", 31, 129, 1281, 23),   # in the forward only
    ("FP32", 15, 64, 128, 4), ("FP32", 15, 17, 65, 2), ("FP32", 43, 100, 63, 3),
])
def test_small_tiles_equal_large_ones(prec, K, h, w, n):
    from paper_2302_05804_amd import em
    p = synth.make_problem("c2", H=h, W=w, n=n, K=K, seed=740 + h)
    code = getattr(em, prec)
    log(f"{prec} K={K} {h}x{w} n={n}")
    a, _ = gpu_run(p.y, p.v, p.psf, 1, 3, x0=None, precision=code, trace=False)
    srv = em.Server(256 << 20, max_slots=2)
    jid = srv.submit(em.Problem.make(n, h, w, K, precision=code), p.y, p.v, p.psf, 3)
    b, _ = srv.wait(jid)
    srv.close()
    assert np.isfinite(a).all() and np.array_equal(a.astype(np.float32), b)
