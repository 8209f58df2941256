"""Tiles of 16 rows with and without bump values in the solve's update passes:
bumps that cover a corner of the points, all of them or none, with 2, 17 and 66
tiles per wavefront (64 flags are read at a time; one block, so that the tiles
without bumps are left out), against the same solve with one tile per wavefront,
which reads all of F.  The two differ in the order of sums only: LML within
1e-9 relative, gradient within eps cond(A) of its largest component, where
cond(A) <= n n1 / noise = 8.4e6 at the largest case: 2e-9."""
import numpy as np
import pytest

from paper_2205_09070_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65, 100, 1040, 4200])
@pytest.mark.parametrize("cover", ["corner", "all", "none"])
@pytest.mark.parametrize("n1", [3, 16, 20])
def test_tiles_without_bumps(n, cover, n1):
    gu.need_gpu()
    import paper_2205_09070_amd as sd
    w = wl.random_small(n, 3, n1, 1, 17, per_row=10.0, noise_var=1e-2)
    p = wl.unpack_hyper(w.desc, w.h)
    rng = np.random.default_rng(n)
    c = {"corner": 0.15 * rng.random(p["c"].shape), "all": 0.5 + 0.0 * p["c"], "none": 9.0 + p["c"]}[cover]
    r = np.full_like(p["r"], {"corner": 0.1, "all": 1.2, "none": 0.1}[cover])
    h = wl.pack_hyper(w.desc, p["sigma2"], p["r_core"], p["a"], p["beta"], r, c, p["noise_var"])
    gu.log("bump tiles n=%d %s n1=%d" % (n, cover, n1))
    est = sd.estimator(probes=5, seed=5, cg_rtol=1e-12, cg_max_iter=4000, precond=1, operator_form=1)
    out = []
    for blocks in (1, 128):
        ctx = gu.ctx()
        ctx.set_option("update_blocks", blocks)   # the block CG at every n
        out.append(ctx.lml_grad(w.desc, gu.dev(w.x), gu.dev(w.y), h, est))
    (v, g, i), (v0, g0, i0) = out
    assert abs(i.cg_iters - i0.cg_iters) <= 2
    assert abs(v - v0) <= 1e-9 * max(abs(v0), 1.0)
    assert np.abs(g - g0).max() <= 2e-9 * np.abs(g0).max()
