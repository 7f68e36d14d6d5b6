"""A NaN, an infinity or a value past the working precision anywhere in f ends a refinement
as non-finite, in every kernel that takes the update norms (needs an MI355X)."""
import numpy as np
import pytest

from workloads import normal_noise

pytestmark = pytest.mark.gpu

ENONFINITE = 6
VALUES = [np.nan, np.inf, -np.inf, 1e300]
# FP32: planes in one block, separate strips, rotating passes; BF16: each block tile's unfold
MESHES = [("f32", 4, (4, 5, 6)), ("f32", 4, (26, 21, 30)), ("f32", 4, (257, 2, 3)), ("bf16", 3, (9, 8, 11)),
          ("bf16x3", 5, (9, 8, 30)), ("bf16x3", 4, (3, 130, 70))]


@pytest.mark.parametrize("prec,k,ne", MESHES)
def test_single_solve(prec, k, ne):
    import torch
    import paper_2310_00226_amd as P
    plan = P.Plan(k, ne, (-1, 1) * 3, 1.0, "dirichlet")
    clean = torch.from_numpy(normal_noise(plan.shape, seed=3)).cuda()
    want = plan.solve(clean)
    for value in VALUES:
        for at in (0, plan.numel - 1, plan.numel // 2):
            f = clean.clone()
            f.view(-1)[at] = value
            u, it, rel, st = plan.solve_refined(f, prec=prec, tol=1e-11, raise_on_error=False)
            assert (st, it) == (ENONFINITE, 1), (value, at)
    u, it, rel, st = plan.solve_refined(clean, prec=prec, tol=1e-11)  # nothing is left behind
    assert st == 0 and float((u - want).abs().max()) <= 1e-10 * float(want.abs().max())


@pytest.mark.parametrize("prec", ["f32", "bf16x3"])
@pytest.mark.parametrize("bad", [0, 1, 2, 3])
def test_batch(prec, bad):
    """One of a small, an ordinary, a solo and a repeated problem: the others converge."""
    import torch
    import paper_2310_00226_amd as P
    plans = [P.Plan(k, ne, (-1, 1) * 3, 1.0, "dirichlet") for k, ne in ((3, (4, 5, 3)), (4, (20, 22, 19)), (4, (26, 27, 26)))]
    plans.append(plans[1])
    fs = [torch.from_numpy(normal_noise(p.shape, seed=9 + i)).cuda() for i, p in enumerate(plans)]
    wants = [p.solve(f) for p, f in zip(plans, fs)]
    batch = P.Batch(plans)
    for value in VALUES:
        gs = [f.clone() for f in fs]
        gs[bad].view(-1)[-1] = value
        us = [torch.empty_like(f) for f in fs]
        its, st = batch.solve(gs, us, prec=prec, tol=1e-11, raise_on_error=False)
        assert st == ENONFINITE and its[bad] == 1, value
        for i in range(4):
            if i != bad:
                assert float((us[i] - wants[i]).abs().max()) <= 1e-10 * float(wants[i].abs().max()), (value, i)
