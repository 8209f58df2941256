"""Canonical CSR: rows of 1, about 64, 511, 512, 513 and 1500 entries (a
wavefront ranks up to 512; one longer row sends all rows to the segmented
sort), against the sorted-order assembly mapped by its permutation: columns,
row pointers and values are the same to the bit, and columns ascend."""
import numpy as np
import pytest
import scipy.sparse as ssp

from paper_2205_09070_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,per_row", [(1, 1.0), (63, 5.0), (3000, 1.0), (3000, 64.0), (511, 1e5), (512, 1e5),
                                       (513, 1e5), (1500, 1e5), (3000, 900.0)])
def test_rows_ascend(n, per_row):
    gu.need_gpu()
    w = wl.random_small(max(n, 2), 2, 2, 2, 8, per_row=per_row)
    gu.log("canonical n=%d per_row %g" % (n, per_row))
    x = gu.dev(w.x[:n])
    c = gu.ctx()
    rp, col, val = (t.cpu().numpy() for t in c.kernel_assemble(w.desc, x, w.h))
    srp, scol, sval, perm = (t.cpu().numpy() for t in c.kernel_assemble(w.desc, x, w.h, sorted_order=True))
    gu.log("  entries %d, longest row %d" % (len(col), np.diff(rp).max()))
    rows = perm[np.repeat(np.arange(n), np.diff(srp))]
    order = np.lexsort((perm[scol], rows))
    assert c.kernel_nnz(w.desc, x, w.h) == rp[-1] == len(order)
    assert (rp == np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))])).all()
    assert (col == perm[scol][order]).all() and (val == sval[order]).all()
