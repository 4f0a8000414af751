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


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("width", [1, 2])
def test_plane_major_zeros_have_the_sign_of_point_major(dtype, width):
    """Rows whose sums cancel, copies of +0 and rows without entries, under
    every component rotation: the sign applies to the sum, so a negated
    component is -0, in both layouts."""
    dt, tdt = (hb.F64, torch.float64) if dtype == "f64" else (hb.F32, torch.float32)
    rots = [(s, 0, 0, t) for s in (1, -1) for t in (1, -1)] + [(0, s, t, 0) for s in (1, -1) for t in (1, -1)]
    n, I, vec = 8 * 3 + 2, 6, (2, 2, 2)
    g = hb.Grid([0], [n])
    g.add_block([(0, n)], [(24, 26)])
    p = hb.Program(g)
    neg = torch.zeros(n, I, dtype=torch.bool)
    for k, r in enumerate(rots):
        if width == 1:
            p.add_ell([(k, k + 1)], 1, [24], [2.0], rot=r)
        else:
            p.add_ell([(k, k + 1)], 2, [24, 25], [1.0, -1.0], rot=r)
        p.add_map([(8 + k, 9 + k)], [[0]], [24], rot=r)
        p.add_csr([(16 + k, 17 + k)], [0, 0], [], [], rot=r)
        for a, s in enumerate((r[0] + r[1], r[2] + r[3])):
            for row in (k, 8 + k, 16 + k):
                neg[row, 2 + 2 * a:4 + 2 * a] = s < 0
    x = torch.full((n, I), 3.0)
    x[24:] = 0.0 if width == 1 else 1.0  # copies of 1 need no sign of zero: only the sums cancel
    zero = torch.zeros(n, dtype=torch.bool)
    zero[:24] = True
    if width == 2:
        zero[8:16] = False
    point, plane = x.to(tdt).cuda(), x.t().contiguous().to(tdt).cuda()
    hb.apply(hb.Plan(p, inner=I, vec=vec, dtype=dt), point)
    hb.apply(hb.Plan(p, inner=I, vec=vec, dtype=dt, order=hb.PLANE_MAJOR), plane)
    torch.cuda.synchronize()
    for got in (point.cpu(), plane.t().cpu()):
        assert (got[zero] == 0).all()
        assert torch.equal(torch.signbit(got[zero]), neg[zero])
