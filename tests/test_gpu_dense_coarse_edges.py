"""The dense coarse factorisation at its smallest numbers of 64-row tile
columns: it takes two a step, looks two ahead and leaves a last single one.
Against the oracle's coarse term with the bar of the other parity tests,
max(1e-10, 10 F), F the oracle's own floor under a reversed local order."""
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


@pytest.mark.parametrize("nparts", [5, 16, 17, 40, 64, 70, 85])  # 1, 1, 2, 3, 4, 5, 6 tile columns
def test_dense_coarse_small_tile_counts(nparts):
    k = np.exp(np.random.default_rng(101).standard_normal((4 * nparts, 10)))
    A = darcy.tpfa_matrix(k)
    part = (np.arange(4 * nparts)[:, None] // 4 + np.zeros(10, int)).astype(np.int32).ravel()
    M = A.to_scipy()
    st = O.setup(M, part, nparts, 4, 1)
    alt = O.setup(M, part, nparts, 4, 1, local_order="descending")
    print("dense coarse", nparts, st.nc, file=sys.stderr, flush=True)
    pc = P.setup(A, part, nparts, 4, overlap=1, coarse_solver="dense")
    r = np.random.default_rng(102).standard_normal(A.n)
    z = pc.apply(torch.tensor(r, device="cuda"), parts=2)
    torch.cuda.synchronize()
    z = z.cpu().numpy()
    pc.close()
    ref, other = O.coarse_part(st, r), O.coarse_part(alt, r)
    floor = np.linalg.norm(other - ref) / np.linalg.norm(ref)
    err = np.linalg.norm(z - ref) / np.linalg.norm(ref)
    print("  err", err, "floor", floor, file=sys.stderr, flush=True)
    assert err <= max(1e-10, 10 * floor)
