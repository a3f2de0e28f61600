"""The sparse coarse solve's launch variants (a whole tile or a quarter per
workgroup, four or sixteen wavefronts, one column or several at once) on a
three-dimensional tree whose root front has more than sixteen tiles, against
the oracle's dense coarse term.  Bar: max(1e-10, 10 F) with F the oracle's own
floor under a rounding-only change (reversed local order)."""
import sys

import numpy as np
import pytest

import oracle as O
from workloads import darcy

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2606_04864_amd as P  # noqa: E402

_C = {}


def case():
    if not _C:
        k = np.exp(np.random.default_rng(71).standard_normal((24, 24, 24)))
        A = darcy.tpfa_matrix(k, 0.1 * k)
        at = np.arange(24) // 3
        part = (at[:, None, None] * 64 + at[:, None] * 8 + at).astype(np.int32).ravel()
        M = A.to_scipy()
        _C["x"] = (A, part, O.setup(M, part, 512, 10, 1),
                   O.setup(M, part, 512, 10, 1, local_order="descending"))
    return _C["x"]


@pytest.mark.parametrize("cols", [1, 5, 16])
def test_tree_solve_variants(cols):
    A, part, st, alt = case()
    pc = P.setup(A, part, 512, 10, overlap=1, coarse_solver="sparse")
    print("tree solve", cols, pc.info["coarse_fronts"], pc.info["coarse_levels"], file=sys.stderr,
          flush=True)
    R = np.random.default_rng(72).standard_normal((cols, A.n))
    Z = pc.apply_columns(torch.tensor(R, device="cuda"), parts=2)
    torch.cuda.synchronize()
    Z = Z.cpu().numpy()
    pc.close()
    for j in range(cols):
        ref = O.coarse_part(st, R[j])
        floor = np.linalg.norm(O.coarse_part(alt, R[j]) - ref) / np.linalg.norm(ref)
        err = np.linalg.norm(Z[j] - ref) / np.linalg.norm(ref)
        assert err <= max(1e-10, 10 * floor), (j, err, floor)
