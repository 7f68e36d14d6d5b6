"""Device memory of a plan: the factors that its solves read, each once (needs an MI355X)."""
import gc

import pytest

pytestmark = pytest.mark.gpu

MB = 1 << 20


def _used(torch, step):
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    out = step()
    torch.cuda.synchronize()
    return out, before - torch.cuda.mem_get_info()[0]


def test_plan_holds_one_copy_of_the_fp64_factors():
    """1023 nodes an axis (nrep = 512): F and S of 1024^2, and the four half-size blocks in
    the strips' order; another copy of those for the tile kernels would be 10 MiB an axis.
    12 MiB for the vectors and the allocations' granularity."""
    import torch
    import paper_2310_00226_amd as P
    P.Plan(1, (4, 4, 4), (-1, 1) * 3, 1.0, "dirichlet").solve(torch.ones((3, 3, 3), dtype=torch.float64, device="cuda"))
    gc.collect()
    plan, used = _used(torch, lambda: P.Plan(1, (1024, 1024, 1024), (-1, 1) * 3, 1.0, "dirichlet"))
    dense, strips = 2 * 1024 * 1024 * 8, 4 * (512 + 32) * 512 * 8
    assert plan.shape == (1023,) * 3 and 0 < used <= 3 * (dense + strips) + 12 * MB, used / MB
