"""The update norms of the refinement (max|delta|, max|u| spread over slots by the
blocks of the last pass) equal the norms of the arrays themselves (needs an MI355X)."""
import numpy as np
import pytest

from workloads import normal_noise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "bf16", "bf16x3"])
# one block; fewer blocks than slots; many blocks, the maximum in the last ones
@pytest.mark.parametrize("k,ne", [(2, (2, 2, 2)), (3, (5, 4, 9)), (4, (20, 24, 17))])
def test_last_update_rel_is_the_ratio_of_the_norms(prec, k, ne):
    import torch
    import paper_2310_00226_amd as P
    plan = P.Plan(k, ne, (-1, 1) * 3, 1.0, "dirichlet")
    f = normal_noise(plan.shape, seed=17 + k)
    f[-1, -1, -1] = 500.0
    f = torch.from_numpy(f).cuda()
    us = []
    for its in (1, 2):
        u, it, rel, st = plan.solve_refined(f, prec=prec, tol=0.0, max_iter=its)
        us.append(u.cpu().numpy())
        if its == 1:
            assert it == 1 and rel == 1.0  # u = delta
    want = np.abs(us[1] - us[0]).max() / np.abs(us[1]).max()
    # u2 - u1 is delta up to the rounding of u2: 2^-53 max|u2| absolutely
    assert abs(rel - want) <= 2.0 ** -52 + 1e-12 * want, (rel, want)
