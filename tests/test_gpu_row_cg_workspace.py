"""Device memory of CG on several columns: a call takes no more than four vectors
per column, what column-by-column vectors would be (they are rows of 8 or 16 values inside),
beside the handle's block workspace and small tables."""
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

TABLES = 6 << 20  # partial sums, row blocks and scalars, each rounded up to the allocator's pages


@pytest.mark.parametrize("batched,cols", [(True, 1), (False, 2), (True, 3), (False, 8), (True, 9), (True, 16)])
def test_workspace_per_column(batched, cols):
    A = darcy.tpfa_matrix(log_field((512, 512), 31))
    pc = P.setup(A, box_partition(512, 512, 16, 16), 256, 4, overlap=1, precision="fp32")
    F = torch.tensor(np.random.default_rng(32).standard_normal((cols, A.n)), device="cuda")
    Ft = F.t().contiguous()
    u = torch.empty_like(F)
    pc.apply_columns(torch.cat([F, F]))  # the block workspace and the factor's copy
    if batched:
        pc.pcg_batched(Ft, [0, A.n], 1e-6, 500)  # torch's own temporaries
    print("row cg workspace", batched, cols, file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    P._lib.amsp_release_caches()
    before = torch.cuda.mem_get_info()[0]
    if batched:
        pc.pcg_batched(Ft, [0, A.n], 1e-6, 500)
    else:
        pc.pcg_columns(F, 1e-6, 500, out=u)
    torch.cuda.synchronize()
    used = before - torch.cuda.mem_get_info()[0]
    pc.close()
    print("  used", used, "of", 32 * A.n * cols + TABLES, file=sys.stderr, flush=True)
    assert used <= 32 * A.n * cols + TABLES
