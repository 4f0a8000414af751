"""What an autotuned shape is stored under, and which shapes are tried."""
import json

import pytest

from helpers import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch

    import paper_2605_14780_amd as hb


def tuned(plan, path):
    fields = [torch.zeros(plan.nelem, device="cuda", dtype=torch.float64 if plan.dtype == hb.F64 else torch.float32)
              for _ in range(2)]
    plan.autotune(fields, cache_path=str(path))
    return [json.loads(line)["key"] for line in open(path)]


def test_plans_served_by_other_kernels_store_their_own_shapes(tmp_path):
    """The same rows in window runs (of a fixed length, or tuned), in the row
    kernel, with b: a shape tuned for one says nothing about another."""
    N, h = 24, 2
    path = tmp_path / "tune.jsonl"
    for inner in (33, 64):
        plain = hb.cs_program(N, h, hb.CS_LAGRANGE)[1]
        with_b = hb.cs_program(N, h, hb.CS_LAGRANGE)[1]
        with_b.add_vector([(0, 1), (0, N), (-h, 0)], [1.0] * (N * h))
        for prog in (plain, with_b):
            for windows in (True, False):
                keys = tuned(hb.Plan(prog, inner=inner, windows=windows), path)
    assert len(keys) == len(set(keys)) == 8


@pytest.mark.parametrize("rows,inner,order", [("lagrange", 33, 0), ("quad", 64, 0), ("quad", 2, 0)])
def test_plans_whose_shape_cuts_corners_only_keep_it(tmp_path, rows, inner, order):
    """Rows in fixed runs, wide or narrow tiles take no launch shape: the
    default stays, whatever the timings of shapes that change nothing."""
    p = hb.Program(hb.Grid.cubed_sphere(24, 2))
    if rows == "quad":
        p.cs_add_quadrature(24, 2, 2)
    else:
        p = hb.cs_program(24, 2, hb.CS_LAGRANGE)[1]
    plan = hb.Plan(p, inner=inner, order=order)
    default = plan.tune
    assert len(tuned(plan, tmp_path / "tune.jsonl")) == 1
    assert plan.tune == default


@pytest.mark.parametrize("mode,inner", [("lagrange", 1), ("sync", 64), ("lagrange", 40)])
def test_plane_pieces_keep_lanes_and_rows(tmp_path, mode, inner):
    p = hb.cs_program(24, 2, hb.CS_LAGRANGE if mode == "lagrange" else hb.CS_SYNC)[1]
    plan = hb.Plan(p, inner=inner, order=hb.PLANE_MAJOR)
    default = plan.tune
    tuned(plan, tmp_path / "tune.jsonl")
    assert [plan.tune[k] for k in ("lanes_per_row", "rows_per_tile")] == [default[k] for k in ("lanes_per_row", "rows_per_tile")]


def test_short_window_rows_are_tried_in_one_order(tmp_path):
    """Rows of at most 32 vectors have one order of loads and stores."""
    plan = hb.Plan(hb.cs_program(48, 3, hb.CS_LAGRANGE)[1], inner=64)
    tuned(plan, tmp_path / "tune.jsonl")
    assert plan.tune["window_order"] == 0
