"""Step lengths of the conjugate gradients on the device: every route of the inner
products against the oracle, and a breakdown leaves the last good iterate (needs an
MI355X)."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

BOX = (-1.0, 1.0, 0.0, 1.5, -0.5, 0.5)


def _problem(k, ne, vmin, vmax):
    import torch
    import paper_2310_00226_amd as P
    prob, plan = O.Problem(k, ne, BOX, 1.0, "dirichlet"), P.Plan(k, ne, BOX, 1.0, "dirichlet")
    rng = np.random.default_rng(17)
    v, f = rng.uniform(vmin, vmax, size=prob.shape), rng.standard_normal(prob.shape)
    return prob, plan, v, f, torch.from_numpy(v).cuda(), torch.from_numpy(f).cuda()


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16x3"])
@pytest.mark.parametrize("k,ne", [(9, (2, 3, 4)), (1, (2, 2, 2)), (1, (3, 90, 60))])
def test_oracle(k, ne, prec):
    """Without and with <p, q> from the march, one node and more partial sums than threads."""
    prob, plan, v, f, vd, fd = _problem(k, ne, 0.0, 10.0)
    ref, _, _ = O.pcg_schrodinger(prob, v, f, 6.0, tol=1e-14, max_iter=300)
    u, _, rel, st = plan.pcg_solve(vd, fd, shift=6.0, prec=prec, tol=1e-13, max_iter=300)
    assert st == 0 and rel <= 1e-13
    assert O.rel_max_err(u.cpu().numpy(), ref) <= 1e-10


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16x3"])
@pytest.mark.parametrize("k,vmin,vmax", [(4, -1e6, -1e5), (4, -120.0, 0.0), (9, -120.0, 0.0)])
def test_breakdown(k, vmin, vmax, prec):
    import torch
    _, plan, _, _, vd, fd = _problem(k, (3, 4, 3), vmin, vmax)

    def run(max_iter):
        return plan.pcg_solve(vd, fd, shift=1.0, prec=prec, tol=1e-13, max_iter=max_iter, raise_on_error=False)
    u, it, rel, st = run(300)
    assert st != 0 and it < 300
    if it == 0:
        assert float(u.abs().max()) == 0.0
        return
    w, jt, rel2, st = run(it)
    assert st != 0 and jt == it and rel2 == rel
    assert torch.equal(u, w)
