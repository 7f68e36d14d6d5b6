"""The residual march on short chunks of x (grids of few blocks), chunks that do not
divide the axis and axes of fewer planes than a chunk (needs an MI355X)."""
import numpy as np
import pytest

import oracle as O
from workloads import normal_noise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,ne,bc", [(1, (70, 9, 9), "dirichlet"), (4, (30, 8, 8), "periodic"),
                                     (5, (23, 24, 24), "dirichlet"), (8, (25, 25, 15), "neumann"),
                                     (7, (1, 40, 3), "dirichlet"), (2, (5, 60, 70), "periodic")])
def test_residual(k, ne, bc):
    import torch
    import paper_2310_00226_amd as P
    box, alpha = (-1, 1, 0, 2, -1, 1), 0.75
    prob, plan = O.Problem(k, ne, box, alpha, bc), P.Plan(k, ne, box, alpha, bc)
    u, f = normal_noise(prob.shape, seed=31), normal_noise(prob.shape, seed=32)
    r = plan.residual(torch.from_numpy(u).cuda(), torch.from_numpy(f).cuda()).cpu().numpy()
    hnorm = sum(np.max(np.sum(np.abs(prob.h_dense(a)), axis=1)) for a in range(3)) + alpha
    assert np.max(np.abs(r - O.residual(prob, u, f))) <= 1e-14 * hnorm


@pytest.mark.parametrize("k,ne,bc", [(3, (70, 60, 50), "neumann"), (6, (9, 30, 26), "periodic"), (8, (4, 3, 17), "neumann")])
def test_residual_rows(k, ne, bc):
    """Two rows of y per wave (large grids, k < 6) and one, ragged in y and z."""
    test_residual(k, ne, bc)


@pytest.mark.parametrize("k,ne,bc", [(4, (64, 64, 64), "neumann"), (7, (30, 30, 30), "dirichlet"), (5, (3, 90, 90), "periodic")])
def test_residual_rounds(k, ne, bc):
    """Chunks of one full round of blocks, of two, and more columns than a round has."""
    test_residual(k, ne, bc)
