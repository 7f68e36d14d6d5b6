"""Axes past 1024 nodes, whose products run on the FP64 tiles and the FP32 rotating passes
instead of the strips (needs an MI355X)."""
import numpy as np
import pytest

import oracle as O
from workloads import normal_noise

pytestmark = pytest.mark.gpu

D, N, C = "dirichlet", "neumann", "periodic"
BOX = (-1, 1, 0, 1.5, -1, 2)
AXES = [(0,), (1,), (2,), (0, 1), (0, 2), (1, 2)]


def _mesh(axes):
    """k = 4: 1027 (Dirichlet), 1029 (Neumann) or 1028 nodes (periodic) on these axes."""
    ne = [2, 1, 3]
    for a in axes:
        ne[a] = 257
    return tuple(ne)


def _floor(prob, lam, g, f, want):
    """Rounding floor of the oracle: the axes contracted in another order."""
    t = f
    for a in (0, 1, 2):
        t = O.mode_product(t, prob.eig[a][2], a)
    t = t * g(lam)
    for a in (0, 1, 2):
        t = O.mode_product(t, prob.eig[a][1], a)
    return np.max(np.abs(t - want))


@pytest.mark.parametrize("axes", AXES)
@pytest.mark.parametrize("bc", [D, C, (C, N, D), (N, D, C)], ids=str)
def test_fp64_tiles(axes, bc):
    """Solve, exponential and power (1e-12 + 10 x the oracle's floor, as for every FP64
    solve), each also in place and without allocation, bit for bit."""
    import torch
    import paper_2310_00226_amd as P
    ne = _mesh(axes)
    prob, plan = O.Problem(4, ne, BOX, 1.25, bc), P.Plan(4, ne, BOX, 1.25, bc)
    f = normal_noise(prob.shape, seed=61)
    fd = torch.from_numpy(f).cuda()
    calls = [(lambda x, u: plan.solve(x, u), lambda s: 1 / s, O.fd_solve(prob, f))]
    for kind, param, g in (("exp", 1e-3, lambda s: np.exp(-1e-3 * s)), ("power", 0.75, lambda s: s ** -0.75)):
        calls.append((lambda x, u, kind=kind, param=param: plan.apply_spectral(kind, 1.25, param, x, u), g,
                      O.spectral_apply(prob, kind, 1.25, param, f)))
    lam = prob.lam3() + 1.25
    for i, (call, g, want) in enumerate(calls):
        u = call(fd, torch.empty_like(fd))
        assert torch.equal(fd.cpu(), torch.from_numpy(f)), i  # f is read only
        bound = 1e-12 * np.max(np.abs(want)) + 10 * _floor(prob, lam, g, f, want)
        assert np.max(np.abs(u.cpu().numpy() - want)) <= bound, i
        x = fd.clone()
        assert torch.equal(call(x, x), u), i
        if i == 0 and plan.numel <= 1 << 23:
            assert torch.equal(plan.solve_noalloc(fd), u)
            x = fd.clone()
            assert torch.equal(plan.solve_noalloc(x, x), u)


@pytest.mark.parametrize("axes", AXES[:3] + [(0, 2)])
@pytest.mark.parametrize("bc", [D, C, N])
def test_fp32_rotating_passes(axes, bc):
    """The four tile heights give the same bits, and the refined solve meets the bar of
    every refined solve (1e-10 + 10 x the oracle's floor)."""
    import torch
    import paper_2310_00226_amd as P
    ne = _mesh(axes)
    prob, plan = O.Problem(4, ne, BOX, 1.25, bc), P.Plan(4, ne, BOX, 1.25, bc)
    f = normal_noise(prob.shape, seed=62)
    fd = torch.from_numpy(f).cuda()
    ref = None
    for rows in ([128] * 6, [96] * 6, [64] * 6, [32] * 6, [32, 64, 96, 128, 64, 32]):
        plan.set_tuning("f32", rows)
        u = plan.solve_lowp(fd, prec="f32")
        ur, it, _, st = plan.solve_refined(fd, prec="f32", tol=1e-12)
        assert st == 0
        if ref is None:
            ref = (u, ur, it)
        assert torch.equal(u, ref[0]) and torch.equal(ur, ref[1]) and it == ref[2], rows
    want = O.fd_solve(prob, f)
    bound = 1e-10 * np.max(np.abs(want)) + 10 * np.max(np.abs(want - O.fd_solve(prob, f, order=(0, 1, 2))))
    assert np.max(np.abs(ref[1].cpu().numpy() - want)) <= bound
