"""Batches whose solves lie on both sides of the size from which a solve runs by itself
on a side stream, one plan twice among them (needs an MI355X)."""
import numpy as np
import pytest

import oracle as O
from workloads import normal_noise

pytestmark = pytest.mark.gpu
BOX = (-1, 1, 0, 2, -1, 1)


@pytest.mark.parametrize("prec", ["f32", "bf16x3"])
def test_solo_and_persistent(prec):
    import torch
    import paper_2310_00226_amd as P
    # 99^3 (just below 10^6), 100^3, (64, 199, 90), a small one, and 101 x 98 x 119
    meshes = [(4, (25, 25, 25), "dirichlet"), (4, (25, 25, 25), "periodic"), (5, (13, 40, 18), ("neumann", "dirichlet", "periodic")),
              (3, (4, 6, 5), "dirichlet"), (6, (17, 17, 20), "dirichlet")]
    plans = [P.Plan(k, ne, BOX, 1.0, bc) for k, ne, bc in meshes]
    pick = [0, 1, 2, 1, 3, 4, 4]  # plans 1 and 4 twice
    batch = P.Batch([plans[i] for i in pick])
    for trial in range(2):
        fs = [normal_noise(plans[i].shape, seed=70 + 10 * trial + j) for j, i in enumerate(pick)]
        us = [torch.full(plans[i].shape, np.nan, dtype=torch.float64, device="cuda") for i in pick]
        its, st = batch.solve([torch.from_numpy(f).cuda() for f in fs], us, prec=prec, tol=1e-12)
        assert st == 0
        for j, i in enumerate(pick):
            k, ne, bc = meshes[i]
            want = O.fd_solve(O.Problem(k, ne, BOX, 1.0, bc), fs[j])
            assert np.max(np.abs(us[j].cpu().numpy() - want)) <= 1e-10 * np.max(np.abs(want)), (trial, j)
