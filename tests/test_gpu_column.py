"""Column CG (one workgroup per few columns, small point sets).

* At the edges of its size classes (64-row slices, 2048, 4096 and 10048
  points) and of its columns per workgroup (256 columns), the column CG and
  the block CG -- taken when a launch shape of the block CG is asked for --
  solve the same systems to the same tolerance: LML within 1e-9 relative and
  gradient within 1e-7 per component, the bounds of the batched-against-single
  test, whose two solves differ in rounding in the same way.
* Test columns of the posterior on both sides of a chunk of 1023 agree with
  the block CG's (chunks of 64) to the posterior test's tolerances."""
import numpy as np
import pytest

from paper_2205_09070_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _both(n, dim, n1, est, **kw):
    import paper_2205_09070_amd as sd
    w = wl.random_small(max(n, 2), dim, n1, 2, 60 + n % 97, per_row=10.0, noise_var=1e-2, **kw)
    x, y = gu.dev(w.x[:n]), gu.dev(w.y[:n])
    out = []
    for block in (False, True):
        c = gu.ctx()
        if block:
            c.set_option("union_spmm", 0)
        v, g, info = c.lml_grad(w.desc, x, y, w.h, est)
        out.append((v, g, info))
    return out


@pytest.mark.parametrize("n", [1, 3, 63, 64, 65, 129, 2048, 2049, 4096, 4097, 10048, 10049])
@pytest.mark.parametrize("form", [(0, 0, 0), (1, 0, 5), (1, 1, 5)], ids=["plain", "lowrank", "factored"])
def test_column_matches_block(n, form):
    gu.need_gpu()
    import paper_2205_09070_amd as sd
    precond, operator, n1 = form
    gu.log("column vs block n=%d form %s" % (n, form))
    est = sd.estimator(probes=3, seed=5, cg_rtol=1e-12, cg_max_iter=4000, precond=precond, operator_form=operator)
    (v, g, i), (v0, g0, i0) = _both(n, 2, n1 if n1 else 2, est)
    assert i.nnz == i0.nnz and abs(i.cg_iters - i0.cg_iters) <= 2
    assert abs(v - v0) <= 1e-9 * max(abs(v0), 1.0)
    assert gu.grad_close(g, g0, rel=1e-7).all()


@pytest.mark.parametrize("n", [255, 256, 300])
def test_exact_columns_per_group(n):
    """n + 1 columns: 256 (one per workgroup), 257 and 301 (four, ragged)."""
    gu.need_gpu()
    import paper_2205_09070_amd as sd
    gu.log("exact columns n=%d" % n)
    (v, g, i), (v0, g0, i0) = _both(n, 3, 3, sd.exact_estimator())
    assert abs(v - v0) <= 1e-9 * abs(v0)
    assert gu.grad_close(g, g0, rel=1e-7).all()


@pytest.mark.parametrize("n,n0", [(2100, 300), (5000, 300), (900, 1023), (900, 1025)])
def test_posterior_columns(n, n0):
    gu.need_gpu()
    import paper_2205_09070_amd as sd
    w = wl.random_small(n, 2, 2, 2, 3, per_row=12.0, noise_var=1e-2)
    x0 = gu.dev(np.random.default_rng(4).random((n0, 2)))
    gu.log("posterior columns n=%d n0=%d" % (n, n0))
    est = sd.estimator(probes=1, cg_rtol=1e-12, cg_max_iter=4000)
    out = []
    for block in (False, True):
        c = gu.ctx()
        if block:
            c.set_option("union_spmm", 0)
        m, v = c.posterior_mean_var(w.desc, gu.dev(w.x), gu.dev(w.y), w.h, x0, est)
        out.append((m.cpu().numpy(), v.cpu().numpy()))
    (m, v), (m0, v0) = out
    assert np.allclose(m, m0, rtol=1e-8, atol=1e-10 * np.abs(m0).max())
    assert np.allclose(v, v0, rtol=1e-7, atol=1e-9 * np.abs(v0).max())
