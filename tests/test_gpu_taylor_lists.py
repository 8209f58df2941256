"""The Taylor log-det over the union lists (union_spmm = 1; the default for
large point sets) against the oracle's estimator and against the plain
products (union_spmm = 0), at odd row counts around the 16-row group and with
probe counts around the 32-column slab.  Tolerances as in the plain form's
test: alpha 1e-13 relative, the log-det 1e-11 relative or 1e-9."""
import pytest

from oracle import estimators as es
from oracle import kernel as kn
from paper_2205_09070_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 15, 17, 1003])
@pytest.mark.parametrize("probes,terms", [(1, 3), (16, 1), (32, 2), (33, 9), (64, 40)])
def test_taylor_over_union_lists(n, probes, terms):
    gu.need_gpu()
    w = wl.random_small(n, 2, 2, 2, 5, per_row=12.0, noise_var=0.3)
    gu.log("taylor lists n=%d probes=%d terms=%d" % (n, probes, terms))
    want, alpha0 = es.boutsidis_logdet(kn.kernel_matrix(w.desc, w.h, w.x), es.rademacher(99, n, probes), terms)
    for form in (1, 0):
        c = gu.ctx()
        c.set_option("union_spmm", form)
        ld, alpha = c.logdet_taylor(w.desc, gu.dev(w.x), w.h, probes=probes, terms=terms, seed=99)
        assert alpha == pytest.approx(alpha0, rel=1e-13)
        assert ld == pytest.approx(want, rel=1e-11, abs=1e-9)
