"""The local eigenproblems at the edges of their passes' row blocks: regions
of up to 16 rows (solved directly), of one row more, and around one and two
blocks of 128 rows, against the oracle's eigenvalues.  Bar as for the other
eigenvalue tests: 1e-10 absolute (spectrum in [0, 2])."""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2606_04864_amd as P  # noqa: E402


def grid(nx, ny, rng):
    """SPD five-point matrix of random couplings (rows nx apart)."""
    def axis(n):
        return sp.diags([rng.uniform(0.5, 2.0, n - 1)], [1], shape=(n, n)) if n > 1 else sp.csr_matrix((1, 1))
    U = sp.kron(sp.eye(ny), axis(nx)) + sp.kron(axis(ny), sp.eye(nx))
    U = U + U.T
    return sp.diags(0.01 + np.asarray(U.sum(axis=1)).ravel()) - U


@pytest.mark.parametrize("nev", [2, 6])
def test_eigenvalues_at_row_block_edges(nev):
    rng = np.random.default_rng(91)
    shapes = [(4, 4), (17, 1), (3, 5), (127, 1), (16, 8), (43, 3), (16, 16), (257, 1)]
    A = sp.block_diag([grid(nx, ny, rng) for nx, ny in shapes], format="csr")
    A.sort_indices()
    sizes = [nx * ny for nx, ny in shapes]
    part = np.repeat(np.arange(len(sizes)), sizes).astype(np.int32)
    print("eigen edges", nev, sizes, file=sys.stderr, flush=True)
    pc = P.Preconditioner(A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data, part,
                          len(sizes), nev, overlap=1)
    lam = pc.eigenvalues()
    unconverged = pc.info["eig_unconverged"]
    pc.close()
    assert unconverged == 0
    st = O.setup(A, part, len(sizes), nev, 1)
    for i, n in enumerate(sizes):
        ref = st.lam[i]
        assert np.max(np.abs(lam[i, : len(ref)] - ref)) <= 1e-10, (i, n)
