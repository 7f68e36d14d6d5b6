"""The BF16 passes with 128- and 256-row block tiles, every pass of the sequence on each,
at extents that just fill or just exceed a tile (needs an MI355X).

Bar: the refined solve within 1e-10 of the oracle (a wrong element would not contract).
"""
import json
import os
import subprocess
import sys

import numpy as np
import pytest

import oracle as O
from workloads import normal_noise

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
D, C = "dirichlet", "periodic"
BOX = (-1, 1, 0, 1.5, -1, 2)
# extents (k = 1); the passes contract z, y, x, z, y, x, and of each group of six, pass i of
# the i-th mesh takes the tile
TILES = {
    # 65 representatives of 128
    "t128-65": [((74, 6, 130), D), ((6, 130, 72), D), ((130, 145, 6), D), ((130, 7, 130), D), ((6, 129, 131), C),
                ((128, 513, 8), C)],
    # 127 and 128 of 128
    "t128-128": [((68, 6, 253), D), ((6, 254, 75), C), ((255, 131, 6), C), ((129, 6, 255), D), ((6, 252, 143), C),
                 ((254, 516, 10), C)],
    # 129 of 128
    "t128-129": [((52, 6, 257), C), ((6, 258, 53), D), ((257, 112, 7), D), ((88, 6, 256), C), ((7, 257, 84), C),
                 ((257, 351, 8), C)],
    # 129 of 256
    "t256-129": [((107, 141, 258), D), ((135, 258, 107), D), ((258, 492, 6), D), ((441, 6, 256), C),
                 ((6, 256, 426), C), ((256, 488, 49), C)],
    # 255 and 256 of 256
    "t256-256": [((97, 131, 512), D), ((129, 511, 98), D), ((511, 390, 6), C), ((389, 6, 510), C), ((6, 511, 410), D),
                 ((511, 448, 48), C)],
    # 257 of 256
    "t256-257": [((80, 129, 513), C), ((132, 513, 79), C), ((512, 308, 6), C)],
}


def _ne(shape, bc):
    return tuple(n + 1 for n in shape) if bc == D else shape


@pytest.mark.parametrize("shape,bc", [m for group in TILES.values() for m in group], ids=lambda v: str(v))
def test_refined_solve(shape, bc):
    import torch
    import paper_2310_00226_amd as P
    ne = _ne(shape, bc)
    prob, plan = O.Problem(1, ne, BOX, 1.5, bc), P.Plan(1, ne, BOX, 1.5, bc)
    assert plan.shape == shape
    f = normal_noise(prob.shape, seed=43)
    want = O.fd_solve(prob, f)
    for prec in ("bf16x3", "bf16"):
        u, it, rel, st = plan.solve_refined(torch.from_numpy(f).cuda(), prec=prec, tol=1e-12, max_iter=60)
        assert st == 0, prec
        assert np.max(np.abs(u.cpu().numpy() - want)) <= 1e-10 * np.max(np.abs(want)), prec


_CHILD = r"""
import json, sys
sys.path.insert(0, {root!r})
import torch
import paper_2310_00226_amd as P
for ne, bc in json.loads(sys.argv[1]):
    for prec in ("bf16", "bf16x3"):
        P.Plan(1, ne, (-1, 1, 0, 1.5, -1, 2), 1.5, bc).tune(prec)
"""


@pytest.mark.parametrize("tile", ["t128", "t256"])
def test_these_meshes_take_the_tile_in_every_kind_of_pass(tile, tmp_path):
    """As the keys of the tuning cache tell: fold, divide, split and FP32 stores."""
    meshes = [(_ne(*m), m[1]) for name, group in TILES.items() if name.startswith(tile) for m in group]
    path = tmp_path / "tune.json"
    r = subprocess.run([sys.executable, "-c", _CHILD.format(root=ROOT), json.dumps(meshes)],
                       env=dict(os.environ, SEM_TUNE_CACHE=str(path)), capture_output=True, text=True, timeout=170)
    assert r.returncode == 0, r.stderr[-2000:]
    taken = {prec: set() for prec in ("bf16", "bf16x3")}
    for key in json.loads(path.read_text())["entries"]:
        _, prec, epi, col, out, *_, t = key.split("|")
        if t == tile:
            taken[prec].add((epi, col, out))
    assert len(taken["bf16"]) == len(taken["bf16x3"]) == 4, taken
