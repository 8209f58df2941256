"""Both sides of the rule for the flags of F's tiles (9 bump functions and more
with the factored operator, 17 with the assembled one): one update block, which
takes the flags there, against 128, which reads all of F.  Bounds as in the test of
the tiles: LML within 1e-9 relative, gradient within eps n n1 / noise of its
largest component (1040 points, 17 bumps: 4e-10)."""
import numpy as np
import pytest

from paper_2205_09070_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,operator", [(8, 1), (9, 1), (16, 0), (17, 0)])
def test_flags_on_both_sides(n1, operator):
    gu.need_gpu()
    import paper_2205_09070_amd as sd
    w = wl.random_small(1040, 3, n1, 1, 17, per_row=10.0, noise_var=1e-2)
    p = wl.unpack_hyper(w.desc, w.h)
    c = 0.15 * np.random.default_rng(n1).random(p["c"].shape)
    h = wl.pack_hyper(w.desc, p["sigma2"], p["r_core"], p["a"], p["beta"], np.full_like(p["r"], 0.1), c, p["noise_var"])
    gu.log("flag rule n1=%d operator %d" % (n1, operator))
    est = sd.estimator(probes=5, seed=5, cg_rtol=1e-12, cg_max_iter=4000, precond=1, operator_form=operator)
    out = []
    for blocks in (1, 128):
        ctx = gu.ctx()
        ctx.set_option("update_blocks", blocks)
        out.append(ctx.lml_grad(w.desc, gu.dev(w.x), gu.dev(w.y), h, est))
    (v, g, i), (v0, g0, i0) = out
    assert abs(i.cg_iters - i0.cg_iters) <= 2
    assert abs(v - v0) <= 1e-9 * max(abs(v0), 1.0)
    assert np.abs(g - g0).max() <= np.finfo(float).eps * 1040 * n1 / 1e-2 * np.abs(g0).max()
