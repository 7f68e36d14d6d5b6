"""The strip products of mode_strip.hip at the edges of their tiles, planes and axis
lengths, against the oracle (needs an MI355X).

Bar (FP64): 1e-12 ||u||_inf + 10 x the oracle's own rounding floor (two contraction
orders), as for every FP64 solve.
"""
import numpy as np
import pytest

import oracle as O
from workloads import normal_noise

pytestmark = pytest.mark.gpu

D, N, C = "dirichlet", "neumann", "periodic"
BOX = (-1, 1, 0, 1.5, -1, 2)


def _check(k, ne, bc, inplace=False):
    import torch
    import paper_2310_00226_amd as P
    prob = O.Problem(k, ne, BOX, 1.25, bc)
    plan = P.Plan(k, ne, BOX, 1.25, bc)
    assert plan.shape == prob.shape
    f = normal_noise(prob.shape, seed=5 + k)
    want = O.fd_solve(prob, f)
    floor = np.max(np.abs(want - O.fd_solve(prob, f, order=(0, 1, 2))))
    fd = torch.from_numpy(f).cuda()
    u = plan.solve(fd, fd if inplace else None).cpu().numpy()
    err, bound = np.max(np.abs(u - want)), 1e-12 * np.max(np.abs(want)) + 10 * floor
    assert err <= bound, (plan.shape, err, bound)


@pytest.mark.parametrize("n", [1, 2, 3, 15, 16, 17, 31, 32, 33, 34, 63, 65, 95, 96])
@pytest.mark.parametrize("bc", [D, C])
def test_planes_at_tile_edges(n, bc):
    """nrep on both sides of a multiple of 16 and 4; y and z in one launch."""
    ne = n + 1 if bc == D else n
    other = {D: (4, 8), C: (3, 6)}[bc]
    _check(1, (other[0], ne, other[1]), bc, inplace=n % 2 == 0)
    _check(1, (other[1], other[0], ne), bc)
    _check(1, (ne, other[1], other[0]), bc)


@pytest.mark.parametrize("ne,bc", [((5, 49, 49), D), ((5, 50, 49), D), ((97, 98, 99), D), ((96, 95, 98), C), ((97, 33, 161), (D, C, N)),
                                   ((5, 255, 97), (N, D, C)), ((3, 96, 96), N)])
def test_separate_axes_at_strip_edges(ne, bc):
    """The largest plane of one launch and the first past it, odd and even strips."""
    _check(1, ne, bc)


@pytest.mark.parametrize("long_axes", [(0,), (1,), (2,), (0, 1), (0, 2), (1, 2)])
@pytest.mark.parametrize("ne,bc", [(128, D), (128, C), (128, N)])
def test_two_tiles_a_wave(long_axes, ne, bc):
    """nrep = 256 and 257, the last with one tile of modes a wave and the first with two."""
    mesh = [6, 3, 4]
    for a in long_axes:
        mesh[a] = ne
    _check(4, tuple(mesh), bc)


@pytest.mark.parametrize("long_axes", [(0,), (1,), (2,), (0, 1), (0, 2), (1, 2)])
@pytest.mark.parametrize("bc", [D, N])
def test_past_the_strips(long_axes, bc):
    """The last length a strip takes (1023, nrep = 512) and the first of the tiles (1025)
    on every set of axes: the two kinds of products hand over to each other."""
    mesh = [2, 1, 2]
    for a in long_axes:
        mesh[a] = 256
    _check(4, tuple(mesh), bc)


def _check_f32(k, ne, bc):
    """FP32 products inside the refinement: the bar of every refined solve, 1e-10 of the
    oracle (a wrong product would not contract)."""
    import torch
    import paper_2310_00226_amd as P
    prob = O.Problem(k, ne, BOX, 1.25, bc)
    plan = P.Plan(k, ne, BOX, 1.25, bc)
    f = normal_noise(prob.shape, seed=5 + k)
    want = O.fd_solve(prob, f)
    u, it, rel, st = plan.solve_refined(torch.from_numpy(f).cuda(), prec="f32", tol=1e-12)
    assert st == 0 and it <= 6
    assert np.max(np.abs(u.cpu().numpy() - want)) <= 1e-10 * np.max(np.abs(want))


@pytest.mark.parametrize("n", [1, 2, 15, 17, 32, 33, 65, 129])
@pytest.mark.parametrize("bc", [D, C])
def test_f32_planes_and_tiles(n, bc):
    ne = n + 1 if bc == D else n
    a, b = {D: (4, 8), C: (3, 6)}[bc]
    for mesh in ((a, ne, b), (b, a, ne), (ne, b, a)):
        _check_f32(1, mesh, bc)


@pytest.mark.parametrize("ne,bc", [((4, 68, 68), D), ((4, 68, 69), D), ((97, 138, 141), D), ((33, 161, 150), (D, C, N)), ((140, 40, 200), N)])
def test_f32_separate_axes(ne, bc):
    _check_f32(1, ne, bc)


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("ne,bc", [(128, N), (255, D), (256, C), (256, N)])
def test_f32_long_axes(axis, ne, bc):
    """Two tiles a wave (nrep = 257 .. 512), and the first length past the strips."""
    mesh = [6, 3, 4]
    mesh[axis] = ne
    _check_f32(4, tuple(mesh), bc)
