"""Canonical CSR with a clique of 530 rows past the rank sort's 512 entries: as a
quarter of the rows and less (sorted by themselves, the short rows ranked) and as
more (all rows sorted), against the sorted-order assembly to the bit."""
import numpy as np
import pytest

from paper_2205_09070_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [531, 2119, 2120, 40000])
def test_long_rows_among_short_ones(n):
    gu.need_gpu()
    k = 530
    rng = np.random.default_rng(5)
    x = 0.6 + 0.4 * rng.random((n, 2))
    x[rng.permutation(n)[:k]] = 0.25 + 0.01 * rng.random((k, 2))
    d = wl.KernelDesc(2, 1, 1, 0, 1)
    h = wl.pack_hyper(d, 1.0, 0.002 if n > 4000 else 0.02, np.full((1, 1), 0.7), np.ones((1, 1)),
                      np.full((1, 1), 0.05), np.full((1, 1, 2), 0.255), 1e-2)
    gu.log("canonical long rows n=%d" % n)
    c = gu.ctx()
    for rep in range(2):                    # the second call meets the first one's storage
        rp, col, val = (t.cpu().numpy() for t in c.kernel_assemble(d, gu.dev(x), h))
        srp, scol, sval, perm = (t.cpu().numpy() for t in c.kernel_assemble(d, gu.dev(x), h, sorted_order=True))
        assert (np.diff(rp) > 512).sum() == k
        rows = perm[np.repeat(np.arange(n), np.diff(srp))]
        order = np.lexsort((perm[scol], rows))
        assert (rp == np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))])).all()
        assert (col == perm[scol][order]).all() and (val == sval[order]).all()
