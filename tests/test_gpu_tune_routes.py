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


def test_batch_tunes_the_problems_of_its_persistent_launches(torch, P):
    """A problem that runs by itself (10^6 unknowns) has no part in their tile rows."""
    small = [P.Plan(3, (6, 7, 5), BOX, 1.0, "dirichlet"), P.Plan(2, (40, 33, 30), BOX, 2.0, "dirichlet")]
    big = P.Plan(4, (26, 27, 26), BOX, 1.0, "dirichlet")
    rows, before = P.Batch(small).tile_rows(), P.tune_stats()
    both = P.Batch(small + [big])
    after = P.tune_stats()
    assert both.tile_rows() == rows
    assert after["misses"] == before["misses"] and after["entries"] == before["entries"], (before, after)
    alone = P.Batch([big, big])
    assert alone.tile_rows() == [0] * 6 and P.tune_stats() == after
    for batch, plans in ((both, small + [big]), (alone, [big, big])):
        fs = [torch.from_numpy(normal_noise(p.shape, seed=40 + i)).cuda() for i, p in enumerate(plans)]
        us = [torch.empty_like(f) for f in fs]
        assert batch.solve(fs, us, prec="f32", tol=1e-12)[1] == 0
        for p, f, u in zip(plans, fs, us):
            want = p.solve(f)
            assert float((u - want).abs().max()) <= 1e-10 * float(want.abs().max())
