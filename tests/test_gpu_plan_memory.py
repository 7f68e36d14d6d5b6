"""Device memory of a plan: the factors that its solves read, each once (needs an MI355X)."""
import gc

import pytest

pytestmark = pytest.mark.gpu

MB = 1 << 20


def _used(torch, step):
    """What step() returns, and the device memory it left allocated outside torch."""
    def held():
        torch.cuda.synchronize()
        free, total = torch.cuda.mem_get_info()
        return total - free - torch.cuda.memory_reserved()
    before = held()
    out = step()
    return out, held() - before


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


def test_low_precision_factors_are_those_that_solves_read():
    """Two axes of 1023 nodes: dense FP32 (1024 + 96 rows), split-BF16 half-size blocks and
    FP32 strips; dense BF16 factors, which no kernel reads, would be 8 MiB an axis."""
    import torch
    import paper_2310_00226_amd as P
    small = P.Plan(1, (4, 4, 4), (-1, 1) * 3, 1.0, "dirichlet")
    small.solve_lowp(torch.ones(small.shape, dtype=torch.float64, device="cuda"), prec="f32")
    plan = P.Plan(1, (1024, 1024, 4), (-1, 1) * 3, 1.0, "dirichlet")
    f = torch.ones(plan.shape, dtype=torch.float64, device="cuda")
    gc.collect()
    _, used = _used(torch, lambda: plan.solve_lowp(f, prec="f32"))
    dense, blocks, strips = 2 * 1120 * 1024 * 4, 2 * 2 * 1024 * 512 * 2, 4 * (512 + 32) * 512 * 4
    assert 0 < used <= 2 * (dense + blocks + strips) + 10 * MB, used / MB
