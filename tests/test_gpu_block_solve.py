"""The local solves, of several columns (the block solve) and of one, at the
edges of their layout, against the oracle's local solves column by column: regions of one block, segments longer
than the rows kept on chip, blocks with more envelope entries than are staged,
the three-dimensional variant, full triangles.  Bar as for the one-column
apply: max(1e-10, 10 F) with F the oracle's own floor under a rounding-only
change (reversed local order)."""
import sys

import numpy as np
import pytest

import oracle as O
from workloads import darcy
from workloads.configs import box_partition

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2606_04864_amd as P  # noqa: E402


def log_field(shape, seed):
    return np.exp(1.5 * np.random.default_rng(seed).standard_normal(shape))


def problem(name):
    """(A, part, nparts, options)"""
    if name == "one_block":  # 36 .. 49 rows per region
        return darcy.tpfa_matrix(log_field((12, 12), 1)), box_partition(12, 12, 2, 2), 4, {}
    if name == "long_segments":  # natural order, rows 150 apart: beyond the 128 kept rows
        return (darcy.tpfa_matrix(log_field((150, 24), 2)), box_partition(150, 24, 1, 2), 2,
                {"local_order": "natural"})
    if name == "narrow_and_wide":  # blocks of few entries, and of more than are staged
        ix, iy = np.meshgrid(np.arange(170), np.arange(60), indexing="xy")
        part = np.where((ix >= 110) | ((ix >= 4) & (iy >= 20) & (iy < 26)), 0, 1).astype(np.int32)
        return darcy.tpfa_matrix(log_field((170, 60), 3)), part.ravel(), 2, {}
    if name == "cubes":  # 9^3 rows per region
        k = log_field((16, 16, 16), 4)
        at = np.arange(16) // 8
        part = (at[:, None, None] * 4 + at[:, None] * 2 + at).astype(np.int32)
        return darcy.tpfa_matrix(k, 0.1 * k), part.ravel(), 8, {}
    if name == "full_triangles":
        return (darcy.tpfa_matrix(log_field((40, 40), 5)), box_partition(40, 40, 2, 2), 4,
                {"dense_tiles": True})
    raise KeyError(name)


@pytest.mark.parametrize("prec,cols", [("fp64", 3), ("fp32", 3), ("fp64", 1)])
@pytest.mark.parametrize("name", ["one_block", "long_segments", "narrow_and_wide", "cubes",
                                  "full_triangles"])
def test_local_solve_edges(name, prec, cols):
    A, part, nparts, kw = problem(name)
    M = A.to_scipy()
    st = O.setup(M, part, nparts, 2, 1)
    alt = O.setup(M, part, nparts, 2, 1, local_order="descending")
    print("local solve", name, prec, cols, file=sys.stderr, flush=True)
    pc = P.setup(A, part, nparts, 2, overlap=1, precision=prec, **kw)
    R = np.random.default_rng(6).standard_normal((cols, A.n))
    Z = pc.apply_columns(torch.tensor(R, device="cuda"), parts=1)
    torch.cuda.synchronize()
    Z = Z.cpu().numpy()
    pc.close()
    for j in range(cols):
        ref = O.local_part(st, R[j])
        floor = np.linalg.norm(O.local_part(alt, R[j]) - ref) / np.linalg.norm(ref)
        err = np.linalg.norm(Z[j] - ref) / np.linalg.norm(ref)
        # a float32-stored factor: its entries' rounding (6e-8) times the growth that the
        # floor shows for float64's (F / 1.1e-16), at least 1e-5
        bar = max(1e-10, 10 * floor) if prec == "fp64" else max(1e-5, 10 * floor * 6e-8 / 1.1e-16)
        print("  err", err, "bar", bar, file=sys.stderr, flush=True)
        assert err <= bar, (j, err, bar)


@pytest.mark.parametrize("cols", [2, 9])
def test_columns_without_coarse_space(cols):
    """nev = 0 (one-level Schwarz): no basis to read, the coarse part alone is zero."""
    A, part, nparts, _ = problem("one_block")
    st = O.setup(A.to_scipy(), part, nparts, 2, 1)
    pc = P.setup(A, part, nparts, 0, overlap=1)
    print("columns without coarse space", cols, file=sys.stderr, flush=True)
    R = np.random.default_rng(7).standard_normal((cols, A.n))
    Z = pc.apply_columns(torch.tensor(R, device="cuda"))
    Z2 = pc.apply_columns(torch.tensor(R, device="cuda"), parts=2)
    torch.cuda.synchronize()
    Z, Z2 = Z.cpu().numpy(), Z2.cpu().numpy()
    pc.close()
    for j in range(cols):
        ref = O.local_part(st, R[j])
        assert np.linalg.norm(Z[j] - ref) <= 1e-10 * np.linalg.norm(ref)
    assert not Z2.any()


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("name", ["one_block", "long_segments", "narrow_and_wide", "cubes",
                                  "full_triangles", "640", "676"])
def test_mixed_local_apply_edges(name, prec):
    """One vector through the float32 factor: the same edges, and both sides of the number of
    regions from which each region's factor is read as one stream.  Bar as above."""
    if name.isdigit():  # regions of 16 .. 36 rows
        ny, nx = {"640": (20, 32), "676": (26, 26)}[name]
        A = darcy.tpfa_matrix(log_field((4 * ny, 4 * nx), 8))
        at = lambda n: np.arange(4 * n) // 4  # noqa: E731
        part, nparts, kw = (at(ny)[:, None] * nx + at(nx)).astype(np.int32).ravel(), ny * nx, {}
    else:
        A, part, nparts, kw = problem(name)
    M = A.to_scipy()
    st = O.setup(M, part, nparts, 2, 1)
    alt = O.setup(M, part, nparts, 2, 1, local_order="descending")
    print("mixed local apply", name, prec, file=sys.stderr, flush=True)
    pc = P.setup(A, part, nparts, 2, overlap=1, precision=prec, **kw)
    r = np.random.default_rng(9).standard_normal(A.n)
    z = pc.apply(torch.tensor(r, device="cuda"), parts=1)
    torch.cuda.synchronize()
    z = z.cpu().numpy()
    pc.close()
    ref = O.local_part(st, r)
    floor = np.linalg.norm(O.local_part(alt, r) - ref) / np.linalg.norm(ref)
    err = np.linalg.norm(z - ref) / np.linalg.norm(ref)
    bar = max(1e-5, 10 * floor * 6e-8 / 1.1e-16)
    print("  err", err, "bar", bar, file=sys.stderr, flush=True)
    assert err <= bar
