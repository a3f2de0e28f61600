"""The sparse coarse factorisation where its fronts hold one to five tiles (every form of
a level's kernels), against the dense one.  Both solve the same Galerkin system of
condition number below 1e5: float64 to 1e-10, the mixed form's float32 factors (6e-8) to
6e-8 * 1e5."""
import sys

import numpy as np
import pytest

from test_gpu_block_solve import log_field
from workloads import darcy
from workloads.configs import box_partition

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2606_04864_amd as P  # noqa: E402


@pytest.mark.parametrize("prec,bar", [("fp64", 1e-10), ("fp32", 6e-3)])
@pytest.mark.parametrize("bx,by,nev", [(1, 1, 4), (2, 2, 4), (16, 1, 4), (4, 4, 15), (8, 8, 4), (8, 8, 15),
                                       (12, 12, 9), (16, 16, 15)])
def test_small_fronts(bx, by, nev, prec, bar):
    nx, ny = 8 * bx, 8 * by
    A = darcy.tpfa_matrix(log_field((nx, ny), 61) ** 0.5)
    part = box_partition(nx, ny, bx, by)
    print("small fronts", bx, by, nev, prec, file=sys.stderr, flush=True)
    R = torch.tensor(np.random.default_rng(62).standard_normal((3, A.n)), device="cuda")
    z = {}
    for solver in ("dense", "sparse"):
        pc = P.setup(A, part, bx * by, nev, overlap=1, precision=prec, coarse_solver=solver)
        z[solver] = torch.cat([pc.apply(R[0].contiguous(), parts=2)[None],
                               pc.apply_columns(R, parts=2)]).cpu().numpy()
        pc.close()
    for a, b in zip(z["sparse"], z["dense"]):
        err = np.linalg.norm(a - b) / np.linalg.norm(b)
        print("  err", err, "bar", bar, file=sys.stderr, flush=True)
        assert err <= bar
