"""The largest regions that the local apply takes: 10112 padded rows in the FP64 form and
17280 in the mixed ones, one row more being refused.  A chain as one region, without a
coarse space; condition number 9, so a float32 factor's rounding (6e-8) stays below 1e-5
and float64's below 1e-13."""
import sys

import numpy as np
import pytest
import scipy.sparse as sp
from scipy.linalg import solveh_banded

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2606_04864_amd as P  # noqa: E402


def chain(n):
    A = sp.diags([-np.ones(n - 1), np.full(n, 2.5), -np.ones(n - 1)], [-1, 0, 1], format="csr")
    return A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data, np.zeros(n, np.int32), 1, 0


@pytest.mark.parametrize("prec,rows,bar", [("fp64", 10112, 1e-13), ("fp32", 17280, 1e-5)])
def test_largest_region(prec, rows, bar):
    print("largest region", prec, rows, file=sys.stderr, flush=True)
    with pytest.raises(P.AmspError, match="LDS capacity"):
        P.Preconditioner(*chain(rows + 1), overlap=0, precision=prec)
    pc = P.Preconditioner(*chain(rows), overlap=0, precision=prec)
    R = np.random.default_rng(41).standard_normal((3, rows))
    z = pc.apply(torch.tensor(R[0], device="cuda"))
    Z = pc.apply_columns(torch.tensor(R, device="cuda"))
    torch.cuda.synchronize()
    z, Z = z.cpu().numpy(), Z.cpu().numpy()
    pc.close()
    ref = solveh_banded(np.array([np.full(rows, 2.5), np.full(rows, -1.0)]), R.T, lower=True).T
    assert np.linalg.norm(z - ref[0]) <= bar * np.linalg.norm(ref[0])
    for j in range(3):
        assert np.linalg.norm(Z[j] - ref[j]) <= bar * np.linalg.norm(ref[j])
