"""The residual march with two rows of y per wave (grids of at least 384 column chunks,
k < 6) for every k, output format and caller, ragged in y and z, and on planes of more
columns than a round has blocks (needs an MI355X).

Two rows are taken where ceil(nz / 64) ceil(ny / 16) ceil(nx / 8k) >= 384.
"""
import numpy as np
import pytest

import oracle as O
from workloads import normal_noise

pytestmark = pytest.mark.gpu

D, N, C = "dirichlet", "neumann", "periodic"
BOX = (-1, 1, 0, 2, -1, 1)
# (k, elements, conditions): 8 x 16 columns and 3 chunks of x, the last of one plane or a few
TWO_ROWS = [(1, (18, 244, 451), D), (2, (17, 121, 225), N), (3, (17, 81, 150), C), (4, (17, 61, 113), (N, C, D)),
            (5, (17, 49, 90), (C, D, N))]


def _ids(c):
    return f"k{c[0]}"


@pytest.mark.parametrize("k,ne,bc", TWO_ROWS + [
    (1, (9, 370, 962), D),  # 24 x 16 columns, one chunk
    (2, (3, 400, 321), D),  # 50 x 11 columns: more than the 512 blocks of a round
    (5, (2, 163, 129), N),  # 52 x 11
    (7, (1, 58, 101), N),   # 51 x 12 with one row a wave
])
def test_residual(k, ne, bc):
    import torch
    import paper_2310_00226_amd as P
    prob, plan = O.Problem(k, ne, BOX, 0.75, bc, eigen=False), P.Plan(k, ne, BOX, 0.75, bc)
    u, f = normal_noise(prob.shape, seed=31), normal_noise(prob.shape, seed=32)
    r = plan.residual(torch.from_numpy(u).cuda(), torch.from_numpy(f).cuda()).cpu().numpy()
    hnorm = sum(np.max(np.sum(np.abs(prob.h_dense(a)), axis=1)) for a in range(3)) + 0.75
    assert np.max(np.abs(r - O.residual(prob, u, f))) <= 1e-14 * hnorm


@pytest.mark.parametrize("k,ne,bc", TWO_ROWS, ids=lambda v: str(v))
def test_formats_and_weights(k, ne, bc):
    """FP32, BF16 and split-BF16 residuals inside refined solves (1e-10 of the oracle, as
    for every refined solve), and the weighted operator with the fused inner product
    inside PCG."""
    import torch
    import paper_2310_00226_amd as P
    prob, plan = O.Problem(k, ne, BOX, 0.75, bc), P.Plan(k, ne, BOX, 0.75, bc)
    f = normal_noise(prob.shape, seed=33)
    fd = torch.from_numpy(f).cuda()
    want = O.fd_solve(prob, f)
    bound = 1e-10 * np.max(np.abs(want)) + 10 * np.max(np.abs(want - O.fd_solve(prob, f, order=(0, 1, 2))))
    for prec in ("f32", "bf16x3", "bf16"):
        u, it, rel, st = plan.solve_refined(fd, prec=prec, tol=1e-12, max_iter=60)
        assert st == 0 and np.max(np.abs(u.cpu().numpy() - want)) <= bound, prec
    v = np.random.default_rng(34).uniform(0.0, 2.0, prob.shape)
    ref = O.pcg_schrodinger(prob, v, f, 1.75, tol=1e-13, max_iter=60)[0]
    u, it, rel, st = plan.pcg_solve(torch.from_numpy(v).cuda(), fd, shift=1.75, prec="f64", tol=1e-13, max_iter=60)
    assert st == 0 and O.rel_max_err(u.cpu().numpy(), ref) <= 1e-10


def test_batch():
    """Batch entries that stay in the persistent launches and take two rows: thin ones below
    10^6 unknowns, and ones with an axis past 1024 nodes; small ones with one row beside them."""
    import torch
    import paper_2310_00226_amd as P
    meshes = [(1, (3, 370, 962), D), (2, (1, 185, 481), D), (3, (1, 124, 321), D), (4, (1, 93, 257), D),
              (5, (1, 74, 206), N), (3, (5, 4, 7), N), (6, (2, 5, 3), D)]
    probs = [O.Problem(k, ne, BOX, 1.5, bc) for k, ne, bc in meshes]
    plans = [P.Plan(k, ne, BOX, 1.5, bc) for k, ne, bc in meshes]
    fs = [normal_noise(p.shape, seed=50 + i) for i, p in enumerate(probs)]
    us = [torch.full(p.shape, np.nan, dtype=torch.float64, device="cuda") for p in probs]
    its, st = P.Batch(plans).solve([torch.from_numpy(f).cuda() for f in fs], us, prec="f32", tol=1e-12, max_iter=40)
    assert st == 0 and min(its) >= 2
    for i, (prob, f, u) in enumerate(zip(probs, fs, us)):
        want = O.fd_solve(prob, f)
        floor = np.max(np.abs(want - O.fd_solve(prob, f, order=(0, 1, 2))))
        assert np.max(np.abs(u.cpu().numpy() - want)) <= 1e-10 * np.max(np.abs(want)) + 10 * floor, i
