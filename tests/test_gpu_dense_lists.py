"""Union-list SpMM where a batch of 64 list columns holds up to its 1024 values
(rows that share most of their columns; 384 values are loaded at a time): against
the CSR SpMM to the bounds of the test of the two forms."""
import pytest

from paper_2205_09070_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,per_row", [(600, 60.0), (600, 150.0), (601, 300.0), (77, 1e4), (700, 1e4)])
@pytest.mark.parametrize("probes", [3, 40])
def test_dense_batches(n, per_row, probes):
    gu.need_gpu()
    import paper_2205_09070_amd as sd
    w = wl.random_small(n, 2, 3, 2, 70, per_row=per_row, noise_var=1e-1)
    est = sd.estimator(probes=probes, seed=9, cg_rtol=1e-11, cg_max_iter=5000, precond=1)
    out = []
    for union in (1, 0):
        c = gu.ctx()
        c.set_option("union_spmm", union)
        out.append(c.lml_grad(w.desc, gu.dev(w.x), gu.dev(w.y), w.h, est))
        assert c.get_option("last_union_spmm") == union
    (v1, g1, i1), (v0, g0, i0) = out
    gu.log("dense lists n=%d: %.0f entries per row, iterations %d / %d" % (n, i1.nnz / n, i1.cg_iters, i0.cg_iters))
    assert abs(i1.cg_iters - i0.cg_iters) <= 2
    assert abs(v1 - v0) <= 1e-10 * abs(v0)
    assert gu.grad_close(g1, g0, rel=1e-8).all()
