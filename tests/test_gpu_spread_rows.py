"""csr_spmm with odd column counts and 8-byte-aligned operands over few rows of
very different lengths (up to 48 rows a CU: rows far apart in a wavefront, long
ones shared by its four groups) and just past that.  A row's sum of at most 1500
products differs from the oracle's by at most 1500 eps sum |a x|: 3.4e-13.  An
infinite row of X reaches exactly the rows that store an entry for it."""
import numpy as np
import pytest
import scipy.sparse as ssp

from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per_cu,extra", [(12, 1), (12, 1003), (48, 0), (48, 1)])
@pytest.mark.parametrize("R,shift", [(2, 1), (3, 0), (31, 0), (32, 1), (33, 0)])
@pytest.mark.parametrize("long_rows", ["clique", "scattered"])
def test_uneven_rows(per_cu, extra, R, shift, long_rows):
    gu.need_gpu()
    import torch
    n = per_cu * torch.cuda.get_device_properties(0).multi_processor_count + extra
    gu.log("uneven rows n=%d R=%d shift %d %s" % (n, R, shift, long_rows))
    rng = np.random.default_rng(n + R)
    lens = rng.choice([0, 1, 15, 16, 17, 40], n)
    at = np.arange(n // 3, n // 3 + n // 30) if long_rows == "clique" else rng.choice(n, n // 30, replace=False)
    lens[at] = rng.choice([63, 64, 65, 250, 1500], len(at))
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
        err = np.abs(Y - S @ x) - 3.4e-13 * (abs(S) @ np.abs(x))
        assert (err[~hit] <= 0).all()
