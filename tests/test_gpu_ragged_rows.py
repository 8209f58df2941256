"""csr_spmm with odd column counts and 8-byte-aligned operands where four rows
share a wavefront (past 12 rows a CU), on row counts that leave ragged steps and
rows of 0 to 70 entries.  A row's sum of at most 70 products differs from the
oracle's by at most 70 eps sum |a x|: 2e-14.  An infinite row of X reaches exactly
the rows that store an entry for it."""
import numpy as np
import pytest
import scipy.sparse as ssp

from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extra", [0, 1, 2, 1003])
@pytest.mark.parametrize("R,shift", [(2, 1), (3, 0), (17, 0), (31, 0), (32, 1), (33, 0)])
def test_ragged_columns_past_few_rows(extra, R, shift):
    gu.need_gpu()
    import torch
    n = 12 * torch.cuda.get_device_properties(0).multi_processor_count + extra
    gu.log("ragged rows n=%d R=%d shift %d" % (n, R, shift))
    rng = np.random.default_rng(n + R)
    lens = rng.choice([0, 1, 15, 16, 17, 40, 70], n)
    col = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lens]).astype(np.int32)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    val = rng.standard_normal(len(col))
    S = ssp.csr_matrix((val, col, rp), shape=(n, n))
    buf = torch.zeros(n * R + 1, dtype=torch.float64, device="cuda:0")
    X = buf[shift:shift + n * R].view(n, R)
    d = lambda a: torch.from_numpy(a).to("cuda:0")
    for bad in (False, True):
        x = rng.standard_normal((n, R))
        if bad:
            x[0] = np.inf
        X.copy_(d(x))
        Y = gu.ctx().csr_spmm(d(rp), d(col), d(val), X).cpu().numpy()
        hit = np.asarray((S[:, 0] != 0).todense()).ravel() if bad else np.zeros(n, bool)
        assert (np.isinf(Y).all(axis=1) == hit).all()
        x[0] = 0.0 if bad else x[0]
        err = np.abs(Y - S @ x) - 2e-14 * (abs(S) @ np.abs(x))
        assert (err[~hit] <= 0).all()
