"""Equal local eigenvalues are taken in the order of the region's rows: in a region of
eight uncoupled pairs of cells every pair has the eigenvalues 0 and 2, and four
eigenvectors are the constants of the first four pairs."""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2606_04864_amd as P  # noqa: E402


@pytest.mark.parametrize("nev", [1, 4, 7])
def test_ties_in_row_order(nev):
    c = np.array([0.5, 2.0, 1.0, 4.0, 8.0, 0.25, 1.0, 2.0])
    A = sp.block_diag([np.array([[1.25, -1.0], [-1.0, 1.25]]) * x for x in c], format="csr")
    A.sort_indices()
    pc = P.Preconditioner(A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data,
                          np.zeros(16, np.int32), 1, nev, overlap=1, local_order="natural")
    print("eigen ties", nev, file=sys.stderr, flush=True)
    z = pc.apply(torch.ones(16, dtype=torch.float64, device="cuda"), parts=2)
    lam = pc.eigenvalues()[0]
    torch.cuda.synchronize()
    z = z.cpu().numpy().reshape(8, 2)
    pc.close()
    print("  ", lam, z[:, 0], file=sys.stderr, flush=True)
    # a pair's constant: A z = 1 there, its row sums being 0.25 c
    assert np.allclose(z[:nev], (4.0 / c[:nev])[:, None], rtol=1e-12, atol=0)
    assert not z[nev:].any()
