"""CG on several columns and independent problems, at the edges of its row
layout: both row widths (8 and 16) full and not, one column, rows of five and
of nine entries, problems of two rows and of more than one row block that start
inside a 64-row slice, a zero column.  Against dense solves: the residual bar
rtol bounds the solution's error by cond(A) rtol."""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2606_04864_amd as P  # noqa: E402

RTOL = 1e-12


def plane(nx, ny, offsets, rng):
    """SPD matrix of random couplings between plane neighbours."""
    at = np.arange(nx * ny).reshape(ny, nx)
    A = sp.diags(np.full(nx * ny, 0.05)).tolil()
    for dy, dx in offsets:
        for y in range(max(0, -dy), min(ny, ny - dy)):
            for x in range(max(0, -dx), min(nx, nx - dx)):
                i, j, c = at[y, x], at[y + dy, x + dx], rng.uniform(0.5, 2.0)
                A[i, i] += c
                A[j, j] += c
                A[i, j] -= c
                A[j, i] -= c
    return A.tocsr()


@pytest.mark.parametrize("cols", [1, 8, 9, 16])
@pytest.mark.parametrize("offsets", [((0, 1), (1, 0)), ((0, 1), (1, 0), (1, 1), (1, -1))],
                         ids=["five", "nine"])
def test_row_cg_edges(offsets, cols):
    rng = np.random.default_rng(81)
    blocks = [plane(nx, ny, offsets, rng) for nx, ny in ((5, 7), (2, 1), (26, 23), (8, 9))]
    A = sp.block_diag(blocks, format="csr")
    A.sort_indices()
    n = A.shape[0]
    seg = np.concatenate([[0], np.cumsum([b.shape[0] for b in blocks])])
    part = np.concatenate([np.full(35, 0), [1, 1], 2 + (np.arange(598) >= 299), np.full(72, 4)])
    pc = P.Preconditioner(A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data,
                          part.astype(np.int32), 5, 1, overlap=1)
    F = rng.standard_normal((n, cols))
    if cols > 1:
        F[:, cols - 1] = 0.0
    print("row cg", len(offsets), cols, file=sys.stderr, flush=True)
    U, info, its, rel = pc.pcg_batched(torch.tensor(F, device="cuda"), seg, RTOL, 500)
    V, vinfo = pc.pcg(torch.tensor(F, device="cuda"), RTOL, 500)
    torch.cuda.synchronize()
    U, V = U.cpu().numpy(), V.cpu().numpy()
    pc.close()
    assert info["converged"] == 1 and vinfo["converged"] == 1
    assert info["iterations"] == int(np.sum(its)) and rel.shape == (4, cols)
    for s, B in enumerate(blocks):
        D = B.toarray()
        sl = slice(seg[s], seg[s + 1])
        bar = 1.01 * np.linalg.cond(D) * max(RTOL, info["relres_floor"])
        for k in range(cols):
            x = np.linalg.solve(D, F[sl, k])
            assert np.linalg.norm(U[sl, k] - x) <= bar * np.linalg.norm(x), (s, k)
            assert (its[s, k] > 0) == bool(F[sl, k].any())
    D = A.toarray()
    bar = 1.01 * np.linalg.cond(D) * max(RTOL, vinfo["relres_floor"])
    X = np.linalg.solve(D, F)
    for k in range(cols):
        assert np.linalg.norm(V[:, k] - X[:, k]) <= bar * np.linalg.norm(X[:, k]), k
