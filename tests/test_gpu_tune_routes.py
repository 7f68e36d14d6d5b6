"""Launch-shape tuning where several routes exist: only kernels that the solves run are
timed, and their choices are kept apart by route (needs an MI355X)."""
import json
import os
import subprocess
import sys

import numpy as np
import pytest

from workloads import normal_noise

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
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


_CHILD = r"""
import json, sys
sys.path.insert(0, {root!r})
import torch
import paper_2310_00226_amd as P
out = []
for ne in ((72, 37, 130), (67, 36, 177)):
    P.Plan(1, ne, (-1, 1) * 3, 1.0, "dirichlet").tune("bf16x3")
    out.append(P.tune_stats())
print("RESULT " + json.dumps(out), flush=True)
"""


def test_bf16_choices_are_kept_per_block_tile(torch, P, tmp_path):
    """Two plans in the same size buckets; the first pass of the second takes 128-row
    tiles, everything else 64-row ones: its choice is its own."""
    path = tmp_path / "tune.json"
    r = subprocess.run([sys.executable, "-c", _CHILD.format(root=ROOT)], env=dict(os.environ, SEM_TUNE_CACHE=str(path)),
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    first, second = json.loads(r.stdout.split("RESULT ")[1])
    assert first["misses"] == 6 and second["misses"] == 7 and second["hits"] == 5, (first, second)
    tiles = sorted(key.rsplit("|", 1)[1] for key in json.loads(path.read_text())["entries"])
    assert tiles == ["t128"] + ["t64"] * 6
