"""The BF16 passes with each of their block tiles, at sizes where a block of modes or
orbits just fills a tile or just exceeds it (needs an MI355X).

Bar: the refined solve within 1e-10 of the oracle (a wrong element would not contract).
"""
import numpy as np
import pytest

import oracle as O
from workloads import normal_noise

pytestmark = pytest.mark.gpu

D, N, C = "dirichlet", "neumann", "periodic"


# nrep = 64 | 65, 128 | 129, 256 | 257 on each axis, with other axes that make the pass
# take the 64-, 128- or 256-row tile
@pytest.mark.parametrize("ne,bc", [((4, 128, 9), D), ((130, 3, 5), D), ((3, 6, 131), D), ((127, 128, 40), C),
                                   ((40, 257, 127), D), ((254, 12, 30), C), ((512, 8, 5), D), ((7, 5, 514), D),
                                   ((130, 140, 260), (D, N, C)), ((2, 2, 2), N)])
@pytest.mark.parametrize("prec", ["bf16x3", "bf16"])
def test_refined_solve(prec, ne, bc):
    import torch
    import paper_2310_00226_amd as P
    box = (-1, 1, 0, 1.5, -1, 2)
    prob, plan = O.Problem(1, ne, box, 1.5, bc), P.Plan(1, ne, box, 1.5, bc)
    f = normal_noise(prob.shape, seed=41)
    want = O.fd_solve(prob, f)
    u, it, rel, st = plan.solve_refined(torch.from_numpy(f).cuda(), prec=prec, tol=1e-12, max_iter=40)
    assert st == 0
    assert np.max(np.abs(u.cpu().numpy() - want)) <= 1e-10 * np.max(np.abs(want))
