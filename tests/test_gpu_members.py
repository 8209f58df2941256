"""Populations whose members take different solvers, and populations and graph
replays of the block CG (a launch-shape option asks for it, where small point
sets would take the column CG)."""
import numpy as np
import pytest

from paper_2205_09070_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def test_members_on_both_sides_of_the_column_rule():
    """Two members store every pair (block CG), two a few neighbours (column
    CG).  The sparse ones' bits are those of the batch whose dense members are
    invalid, the dense ones' those of a single call (their core radius is the
    population's largest), and all agree with single calls to the bounds of the
    batched-against-single test."""
    gu.need_gpu()
    import paper_2205_09070_amd as sd
    w = wl.random_small(1000, 2, 3, 2, 31, combine=1, per_row=12.0, noise_var=1e-2)
    p = wl.unpack_hyper(w.desc, w.h)
    H = np.array([wl.pack_hyper(w.desc, s2, rc, p["a"], p["beta"], p["r"], p["c"], 0.5)
                  for s2, rc in ((0.7, 2.0), (1.0, p["r_core"]), (0.5, 2.0), (1.2, 0.8 * p["r_core"]))])
    bad = H.copy()
    bad[[0, 2], 0] = -1.0
    est = sd.estimator(probes=8, seed=3, cg_rtol=1e-11, cg_max_iter=3000, precond=1)
    gu.log("members on both sides")
    c = gu.ctx()
    x, y = gu.dev(w.x), gu.dev(w.y)
    v, g, st, info = c.lml_grad_batched(w.desc, x, y, H, est)
    gu.log("  entries %s" % [i.nnz for i in info])
    assert (st == sd.OK).all() and c.get_option("last_update_blocks") > 0
    v1, g1, st1, _ = c.lml_grad_batched(w.desc, x, y, bad, est)
    assert c.get_option("last_update_blocks") == 0
    assert list(st1) == [sd.INVALID_ARG, sd.OK, sd.INVALID_ARG, sd.OK]
    assert np.array_equal(v[1::2], v1[1::2]) and np.array_equal(g[1::2], g1[1::2])
    for m in range(4):
        v1, g1, _ = c.lml_grad(w.desc, x, y, H[m], est)
        assert (c.get_option("last_update_blocks") > 0) == (m % 2 == 0)
        if m % 2 == 0:
            assert v[m] == v1 and np.array_equal(g[m], g1)
        assert abs(v[m] - v1) <= 1e-9 * abs(v1)
        assert gu.grad_close(g[m], g1, rel=1e-7).all()
