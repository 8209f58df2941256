"""Lanczos quadrature on the GPU against z^T ln(A) z from a dense
eigendecomposition, with fewer and with more than the 1024 steps that its
kernel stages at a time: the solves' 1e-12 tolerance leaves the quadrature's
error far below 1e-9 of the log-det."""
import numpy as np
import pytest

from oracle import estimators as es
from oracle import kernel as okn
from paper_2205_09070_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,noise,least", [(1500, 3e-7, 0), (4000, 1e-7, 1025)])
def test_quadrature_of_many_steps(n, noise, least):
    gu.need_gpu()
    import paper_2205_09070_amd as sd
    w = wl.small_2d(n, 3)
    h = w.h.copy()
    h[-1] = noise
    est = sd.estimator(probes=2, seed=11, cg_rtol=1e-12, cg_max_iter=20000)
    v, info = gu.ctx().lml(w.desc, gu.dev(w.x), gu.dev(w.y), h, est)
    lam, Q = np.linalg.eigh(okn.kernel_matrix(w.desc, h, w.x, add_noise=True))
    z = es.rademacher(11, n, 2)
    ld = float(np.mean(np.sum(np.log(lam)[:, None] * (Q.T @ z) ** 2, axis=0)))
    gu.log("steps %d, logdet %.12g dense %.12g" % (info.cg_iters, info.logdet, ld))
    assert info.cg_iters >= least
    assert abs(info.logdet - ld) <= 1e-9 * abs(ld)
