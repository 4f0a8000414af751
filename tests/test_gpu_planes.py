"""Plane-major applies (pieces of rows staged by planes) against point-major
applies of the same program: both take a row's entries in the same order, so
every value is the same bit for bit."""
import numpy as np
import pytest

from helpers import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch

    import paper_2605_14780_amd as hb


# planes: one, a group of 4 less one, whole groups, a remainder; rows: less
# than a run of 64, runs that end inside a block, pieces of 64 to 256 rows;
# the vector's components in whole plane groups, and not
@pytest.mark.parametrize("N,h,I,vec,dtype", [
    (4, 1, 1, None, "f64"), (5, 2, 3, (1, 1, 1), "f64"), (16, 1, 4, None, "f32"), (23, 3, 16, (8, 4, 4), "f64"),
    (21, 2, 22, (2, 10, 10), "f64"), (48, 3, 64, (0, 32, 32), "f32"), (64, 3, 33, None, "f64"),
    (96, 2, 72, (8, 32, 16), "f64")])
@pytest.mark.parametrize("mode", ["sync", "lagrange"])
@pytest.mark.parametrize("ninner", [0, 1, "inner"])
def test_plane_major_matches_point_major(N, h, I, vec, dtype, mode, ninner):
    dt, tdt = (hb.F64, torch.float64) if dtype == "f64" else (hb.F32, torch.float32)
    _, prog = hb.cs_program(N, h, hb.CS_LAGRANGE if mode == "lagrange" else hb.CS_SYNC, vector=vec is not None)
    rng = np.random.default_rng(N + I)
    if ninner:  # b on two strips of every face
        n = I if ninner == "inner" else 1
        for f in range(6):
            prog.add_vector([(f, f + 1), (0, N), (-h, 0)], rng.normal(size=N * h * n), ninner=n)
            prog.add_vector([(f, f + 1), (N, N + h), (0, N)], rng.normal(size=N * h * n), ninner=n)
    x = torch.from_numpy(rng.normal(size=(prog.grid.cells, I))).to(tdt).cuda()
    want = x.clone()
    hb.apply(hb.Plan(prog, inner=I, vec=vec, dtype=dt), want)
    plan = hb.Plan(prog, inner=I, vec=vec, dtype=dt, order=hb.PLANE_MAJOR)
    for tune in (None, dict(block=64, persistent=0), dict(block=192, persistent=5)):
        if tune:
            plan.tune = {**plan.tune, **tune}
        got = x.t().contiguous()
        hb.apply(plan, got)
        torch.cuda.synchronize()
        assert torch.equal(got.t(), want)
