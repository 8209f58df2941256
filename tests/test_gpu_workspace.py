"""Solves near the limits of the workspace they are given."""
import numpy as np
import pytest

from paper_2205_09070_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def test_static_workspace_fits_whatever_the_block_cg_fits():
    """The coefficient histories (16 bytes per iteration and column) bring a
    small solve to the limit of the static workspace: at the last cg_max_iter
    at which the column CG is taken, the rest of the evaluation fits too."""
    gu.need_gpu()
    import paper_2205_09070_amd as sd
    w = wl.random_small(1500, 2, 2, 2, 7, combine=1, per_row=40.0, noise_var=1e-1)
    x, y = gu.dev(w.x), gu.dev(w.y)

    def call(max_iter, block=False):
        c = gu.ctx()
        if block:
            c.set_option("union_spmm", 0)
        est = sd.estimator(probes=1, seed=5, cg_rtol=1e-8, cg_max_iter=max_iter)
        try:
            out = c.lml_grad_noalloc(w.desc, x, y, w.h, est)[0]
        except sd.SdgpError as e:
            assert e.status == sd.OOM, e
            out = None
        return out, c.get_option("last_spmm_blocks") > 0 and c.get_option("last_update_blocks") == 0

    def last(lo, hi, holds):
        while hi - lo > 1:
            mid = (lo + hi) // 2
            lo, hi = (mid, hi) if holds(mid) else (lo, mid)
        return lo

    fits = last(1000, 1 << 23, lambda m: call(m, block=True)[0] is not None)
    column = last(1000, fits + 1, lambda m: call(m)[1])
    gu.log("block CG fits to %d iterations, column CG is taken to %d" % (fits, column))
    assert call(1000)[1] and 1000 < column
    for m in (column, min(column + 1, fits), (column + fits) // 2, fits):
        assert call(m)[0] is not None, m


def test_posterior_keeps_no_coefficients():
    """cg_max_iter bounds the iterations, not the memory, of a posterior whose
    1024 columns are solved together: at 20,000,000 (328 GB if every iteration's
    coefficients had a place) the call gives the bits that it gives at 4000, and
    its last, narrow chunk takes the same solver."""
    gu.need_gpu()
    import paper_2205_09070_amd as sd
    w = wl.random_small(900, 2, 2, 2, 3, per_row=12.0, noise_var=1e-2)
    x, y, x0 = gu.dev(w.x), gu.dev(w.y), gu.dev(np.random.default_rng(4).random((1030, 2)))
    out = []
    for max_iter in (4000, 20_000_000):
        c = gu.ctx()
        m, v = c.posterior_mean_var(w.desc, x, y, w.h, x0, sd.estimator(probes=1, cg_rtol=1e-12, cg_max_iter=max_iter))
        assert c.get_option("last_spmm_blocks") == 7 and c.get_option("last_update_blocks") == 0
        out.append((m.cpu().numpy(), v.cpu().numpy()))
    assert (out[0][0] == out[1][0]).all() and (out[0][1] == out[1][1]).all()
