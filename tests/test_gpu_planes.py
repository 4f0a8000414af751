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


def every_kind(N, h, ninner, vector, pad=0, wide=4):
    """Rows of 22 entries on `wide` of four faces, 4-point rows on the others; copies, 4-point rows, rows of up to 7
    entries, zero rows and b alone on the sides of the other two; b of more values than one padded by `pad`."""
    p = hb.Program(hb.Grid.cubed_sphere(N, h))
    rng = np.random.default_rng(N + h)
    W = N + 2 * h
    eye = np.eye(3, dtype=int)
    rot = (0, -1, 1, 0) if vector else None
    sides = ([(0, N), (-h, 0)], [(0, N), (N, N + h)], [(-h, 0), (0, N)], [(N, N + h), (0, N)])
    for f in range(6):
        for s, box in enumerate(sides):
            rows = [(f, f + 1)] + box
            n = N * h
            kind = "csr" if f < wide else "ell" if f < 4 else ("map", "ell", "ragged", "b")[s] if f == 4 else ("zero", "ell", "csr", "map")[s]
            cells = lambda k: ((f * W + rng.integers(0, N, (n, k)) + h) * W + rng.integers(0, N, (n, k)) + h)  # noqa: E731
            if kind == "csr":
                p.add_csr(rows, np.arange(n + 1) * 22, cells(22), rng.normal(size=(n, 22)), rot=rot)
            elif kind == "ragged":
                k = rng.integers(0, 8, n)
                ptr = np.concatenate([[0], np.cumsum(k)])
                p.add_csr(rows, ptr, cells(7).reshape(-1)[:ptr[-1]], rng.normal(size=ptr[-1]), rot=rot)
            elif kind == "ell":
                p.add_ell(rows, 4, cells(4), rng.normal(size=(n, 4)), rot=rot)
            elif kind == "map":  # the cell across the face
                d = 1 if s >= 2 else 2
                p.add_map(rows, eye, [0] + [(N if box[d - 1][0] < 0 else -N) if k == d else 0 for k in (1, 2)], 0.5,
                          rot=rot)
            elif kind == "zero":
                p.add_zero(rows)
            if kind in ("b", "map", "csr") and f >= 4 and ninner:
                v = np.pad(rng.normal(size=(n, ninner)), ((0, 0), (0, pad if ninner > 1 else 0)))
                p.add_vector(rows, v, ninner=v.shape[1])
    return p


# planes: one, fewer than the sets of a workgroup, uneven shares of the sets,
# groups and a remainder; rows: a part of a tile, several tiles
@pytest.mark.parametrize("N,h,I,vec,dtype,launches", [
    (5, 1, 1, None, "f64", 1), (9, 2, 3, (1, 1, 1), "f64", 1), (8, 3, 9, (0, 4, 4), "f32", 1),
    (24, 2, 16, None, "f64", 1), (13, 2, 33, None, "f32", 1), (10, 3, 64, (16, 16, 16), "f64", 1),
    (7, 2, 100, (0, 50, 50), "f32", 1), (9, 1, 129, None, "f64", 1), (171, 3, 33, (0, 15, 15), "f32", 2)])
@pytest.mark.parametrize("b", [0, 1, "inner"])
def test_plane_major_rows_of_every_kind(N, h, I, vec, dtype, launches, b):
    """One launch serves every row of a plan with rows of many entries (two,
    where many of its rows have few), and gives point-major's bits, in any
    launch shape; its adjoint too, which zeroes them all in one.  (Of rows
    padded to 128 values: point-major sums shorter ones over several lanes.)"""
    dt, tdt = (hb.F64, torch.float64) if dtype == "f64" else (hb.F32, torch.float32)
    ninner, pad = I if b == "inner" else b, max(0, 128 - I)
    wide = 4 if launches == 1 else 1
    p = every_kind(N, h, ninner, vec is not None, wide=wide)
    x = torch.from_numpy(np.random.default_rng(I).normal(size=(p.grid.cells, I))).to(tdt).cuda()
    want = torch.nn.functional.pad(x, (0, pad))
    wanted = want.clone()
    point = hb.Plan(every_kind(N, h, ninner, vec is not None, pad, wide), inner=I + pad, vec=vec, dtype=dt)
    plan = hb.Plan(p, inner=I, vec=vec, dtype=dt, order=hb.PLANE_MAJOR)
    hb.apply(point, want)
    hb.apply_adjoint(point, wanted)
    want, wanted = want[:, :I].contiguous(), wanted[:, :I].contiguous()
    bits = torch.int64 if dtype == "f64" else torch.int32
    for tune in (None, dict(block=64, lanes_per_row=1, rows_per_tile=100), dict(block=192, lanes_per_row=128),
                 dict(block=256, lanes_per_row=32, rows_per_tile=3, persistent=7)):
        if tune:
            plan.tune = {**plan.tune, **tune}
        got = x.t().clone(memory_format=torch.contiguous_format)  # (x itself, of one value a cell)
        hb.apply(plan, got)
        torch.cuda.synchronize()
        assert torch.equal(got.t().contiguous().view(bits), want.view(bits)), tune
        got = x.t().clone(memory_format=torch.contiguous_format)  # (x itself, of one value a cell)
        hb.apply_adjoint(plan, got)
        torch.cuda.synchronize()
        assert torch.equal(got.t(), wanted), tune
    assert len(plan.kernels()) == launches
    assert sum("k_apply" in k for k in plan.kernels(hb.OP_ADJOINT)) == 1
