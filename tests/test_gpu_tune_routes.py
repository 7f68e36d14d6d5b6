"""Launch-shape tuning where several routes exist: only kernels that the solves run are
timed, and their choices are kept apart by route (needs an MI355X)."""
import numpy as np
import pytest

from workloads import normal_noise

pytestmark = pytest.mark.gpu

BOX = (-1, 1, -1, 1, -1, 1)


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


@pytest.fixture(scope="module")
def P():
    import paper_2310_00226_amd as P
    return P


def test_f32_solves_on_strips_time_nothing(torch, P):
    """Axes of up to 1024 nodes: no lookup, no choice, unless a caller asks for one."""
    plan = P.Plan(4, (9, 13, 7), BOX, 1.0, "dirichlet")
    f = torch.from_numpy(normal_noise(plan.shape, seed=5)).cuda()
    before = P.tune_stats()
    plan.solve_lowp(f, prec="f32")
    assert plan.solve_refined(f, prec="f32", tol=1e-11)[3] == 0
    assert plan.pcg_solve(torch.ones_like(f), f, prec="f32", tol=1e-11)[3] == 0
    ch = P.CahnHilliard(4, (9, 13, 7), (0, 6.0) * 3, 0.05, 0.02, 1e-4, prec="f32", refine_sweeps=1)
    assert P.tune_stats() == before
    assert plan.tuning("f32") is None
    assert ch.tuning() == [96 if n <= 96 else 128 for n in ch.shape[::-1]] * 2
    u = plan.solve_lowp(f, prec="f32").cpu().numpy()
    plan.lowp_pass("f32", 0, 1)  # runs a rotating pass, so it picks their shapes
    assert plan.tuning("f32") is not None
    assert np.array_equal(plan.solve_lowp(f, prec="f32").cpu().numpy(), u)


def test_f32_solves_past_the_strips_are_tuned(torch, P):
    plan = P.Plan(4, (2, 257, 3), BOX, 1.0, "dirichlet")
    f = torch.from_numpy(normal_noise(plan.shape, seed=6)).cuda()
    plan.solve_lowp(f, prec="f32")
    assert set(plan.tuning("f32")) <= {128, 96, 64, 32}
