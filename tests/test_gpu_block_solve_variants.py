"""Every instance of the several-column solve (row width 8 and 16, up to 8 and up to 15
eigenvectors, float64 and float32 factor, few and many regions, few and many staged
entries), on the preconditioner itself.

The local solves alone against the oracle's, with the bar of the one-vector solves:
1e-10, with a float32-stored factor its entries' rounding (6e-8) times the growth that the
oracle's own floor under a reversed local order shows, at least 1e-5.  Both parts together
against the two parts alone: a row's sums differ in the order of at most 15 + 8 terms, so by
23 * 1.1e-16 of their size; 1e-12 leaves 400 for their cancellation.  The coarse part against
the one-column one, whose sums run in another order: 1e-10."""
import sys

import numpy as np
import pytest

import oracle as O
from test_gpu_block_solve import log_field, problem
from workloads import darcy
from workloads.configs import box_partition

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2606_04864_amd as P  # noqa: E402


def many_regions():
    """676 regions of 16 .. 36 rows"""
    return darcy.tpfa_matrix(log_field((104, 104), 8)), box_partition(104, 104, 26, 26), 676, {}


@pytest.mark.parametrize("prec,cols", [("fp64", 9), ("fp64", 16), ("fp32", 9), ("fp32", 16), ("bf16", 9)])
@pytest.mark.parametrize("name", ["one_block", "long_segments", "narrow_and_wide", "cubes",
                                  "full_triangles", "many"])
def test_wide_local_solves(name, prec, cols):
    local_solves(name, prec, cols)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_narrow_local_solves_many_regions(prec):
    local_solves("many", prec, 3)


def local_solves(name, prec, cols):
    A, part, nparts, kw = many_regions() if name == "many" else problem(name)
    M = A.to_scipy()
    st = O.setup(M, part, nparts, 2, 1)
    alt = O.setup(M, part, nparts, 2, 1, local_order="descending")
    print("wide local solves", name, prec, cols, file=sys.stderr, flush=True)
    pc = P.setup(A, part, nparts, 2, overlap=1, precision=prec, **kw)
    R = np.random.default_rng(16).standard_normal((cols, A.n))
    Z = pc.apply_columns(torch.tensor(R, device="cuda"), parts=1)
    torch.cuda.synchronize()
    Z = Z.cpu().numpy()
    pc.close()
    for j in range(cols):
        ref = O.local_part(st, R[j])
        floor = np.linalg.norm(O.local_part(alt, R[j]) - ref) / np.linalg.norm(ref)
        err = np.linalg.norm(Z[j] - ref) / np.linalg.norm(ref)
        bar = max(1e-10, 10 * floor) if prec == "fp64" else max(1e-5, 10 * floor * 6e-8 / 1.1e-16)
        assert err <= bar, (j, err, bar)


@pytest.mark.parametrize("cols", [3, 9])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("name,nev", [("one_block", 12), ("cubes", 15), ("cubes", 4), ("many", 9)])
def test_parts_add_up(name, nev, prec, cols):
    A, part, nparts, kw = many_regions() if name == "many" else problem(name)
    print("parts add up", name, nev, prec, cols, file=sys.stderr, flush=True)
    pc = P.setup(A, part, nparts, nev, overlap=1, precision=prec, **kw)
    R = torch.tensor(np.random.default_rng(17).standard_normal((cols, A.n)), device="cuda")
    both, local, coarse = (pc.apply_columns(R, parts=p) for p in (3, 1, 2))
    one = torch.stack([pc.apply(R[j].contiguous(), parts=2) for j in range(cols)])
    torch.cuda.synchronize()
    both, local, coarse, one = (x.cpu().numpy() for x in (both, local, coarse, one))
    pc.close()
    for j in range(cols):
        size = np.linalg.norm(local[j]) + np.linalg.norm(coarse[j])
        assert np.linalg.norm(both[j] - local[j] - coarse[j]) <= 1e-12 * size, j
        assert np.linalg.norm(coarse[j] - one[j]) <= 1e-10 * np.linalg.norm(one[j]), j
        assert np.linalg.norm(coarse[j]) > 0
