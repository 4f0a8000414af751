"""Sliding-window kernel (4-point Lagrange rows of face-edge strips, each
wavefront walking a run of rows along the neighbour's grid line).

Its sum is the general row path's, so the bar is bit identity with a plan of
the same program built with windows=False (the general row kernel), for FP64
and FP32, with and without the component rotation and b, for run lengths from
1 to 64 rows, both orders of loads and stores, and rows of 256 bytes to 2 KiB; the general row path itself is
checked against the oracle elsewhere.  Also: a graph captured before a change
of the launch shape is refused, not replayed over freed tables.
"""
import numpy as np
import pytest

import synthinputs
from helpers import gpu_available
from oracle import cubed_sphere as ocs

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch

    import paper_2605_14780_amd as hb


def cs_pair(N, h, nf, nl, dtype, vector, with_b):
    I = nf * nl
    vec = (2 * nl, nl, nl) if vector else None
    grid, prog = hb.cs_program(N, h, hb.CS_LAGRANGE, vector=vector)
    if with_b:
        rng = np.random.default_rng(N + I)
        for f in (0, 3):
            for side in (ocs.LEFT, ocs.TOP):
                prog.add_vector(ocs.side_box(f, side, N, h), rng.standard_normal((N * h, I)), ninner=I)
        prog.add_vector(ocs.side_box(5, ocs.RIGHT, N, h), rng.standard_normal((N * h, 1)), ninner=1)
    pw = hb.Plan(prog, inner=I, vec=vec, dtype=dtype)
    pr = hb.Plan(prog, inner=I, vec=vec, dtype=dtype, windows=False)
    return grid, pw, pr


def field(N, h, nf, nl, tdt, seed):
    W = N + 2 * h
    I = nf * nl
    full = torch.full((6, W, W, I), float("nan"), dtype=tdt, device="cuda")
    full[:, h:h + N, h:h + N] = synthinputs.cs_sh_field_torch(N, nf, nl, seed=seed, device="cuda").to(tdt)
    return full.reshape(-1)


@pytest.mark.parametrize("N,h,nf,nl,dtype,vector,with_b", [
    (48, 3, 1, 32, "f64", False, False),   # 256-byte rows, the shortest that take windows (without b)
    (40, 3, 4, 16, "f32", True, False),    # 256-byte FP32 rows
    (48, 3, 4, 16, "f64", True, False),    # 512-byte rows
    (48, 3, 4, 16, "f64", True, True),
    (48, 2, 1, 128, "f32", False, True),   # 512-byte FP32 rows
    (96, 3, 4, 32, "f32", True, False),
    (64, 4, 4, 64, "f64", True, True),     # 2 KiB rows, two slices per row
    (37, 3, 4, 24, "f64", True, False),    # odd N, rows of 1.5 slices
    (384, 3, 4, 64, "f64", True, False),   # the C384 workload
    (384, 3, 4, 64, "f32", True, False),
])
def test_window_kernel_bitwise_general_path(N, h, nf, nl, dtype, vector, with_b):
    dt, tdt = (hb.F64, torch.float64) if dtype == "f64" else (hb.F32, torch.float32)
    grid, pw, pr = cs_pair(N, h, nf, nl, dt, vector, with_b)
    st = pw.stats()
    assert st["rows_window"] == st["rows_ell"] > 0 and st["window_runs"] > 0
    assert pr.stats()["rows_window"] == 0
    x = field(N, h, nf, nl, tdt, seed=N)
    want = x.clone()
    hb.apply(pr, want)
    for R in (1, 5, 16, 64):
        for order in (0, 1):  # pipelined and ordered loads and stores
            pw.tune = dict(pw.tune, rows_per_tile=R, window_order=order)
            got = x.clone()
            hb.apply(pw, got)
            torch.cuda.synchronize()
            assert torch.isfinite(got).all(), (R, order)
            assert torch.equal(got, want), (R, order)


def test_window_rows_with_b_from_512_bytes():
    """Segments with b take windows from 512-byte rows, the others from 256:
    at 256 bytes a plan with b on some strips windows only the others, and
    still gives the general path's bits."""
    N, h, nf, nl = 48, 3, 1, 32
    grid, pw, pr = cs_pair(N, h, nf, nl, hb.F64, False, True)
    st = pw.stats()
    assert 0 < st["rows_window"] < st["rows_ell"]
    x = field(N, h, nf, nl, torch.float64, seed=3)
    want, got = x.clone(), x.clone()
    hb.apply(pr, want)
    hb.apply(pw, got)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    grid, pw2, _ = cs_pair(N, h, 4, 16, hb.F64, True, True)  # 512-byte rows: every strip
    st2 = pw2.stats()
    assert st2["rows_window"] == st2["rows_ell"] > 0


def test_window_adjoint_and_graph_after_tuning():
    """The adjoint of a window plan equals the general plan's (same tables);
    a graph captured before set_tune is refused, a new capture runs."""
    N, h, nf, nl = 48, 3, 4, 16
    grid, pw, pr = cs_pair(N, h, nf, nl, hb.F64, True, True)
    gen = torch.Generator(device="cuda").manual_seed(5)
    y = torch.randn(grid.cells * nf * nl, dtype=torch.float64, device="cuda", generator=gen)
    a, b = y.clone(), y.clone()
    hb.apply_adjoint(pw, a)
    hb.apply_adjoint(pr, b)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    x = field(N, h, nf, nl, torch.float64, seed=9)
    want = x.clone()
    hb.apply(pr, want)
    f = x.clone()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        g = hb.ApplyGraph(pw, [f], 2, stream=s.cuda_stream)
        g.launch(s.cuda_stream)
        s.synchronize()
        assert torch.equal(f, want)
        pw.tune = dict(pw.tune, rows_per_tile=7)
        with pytest.raises(hb.HbcError):
            g.launch(s.cuda_stream)
        g2 = hb.ApplyGraph(pw, [f], 2, stream=s.cuda_stream)
        f.copy_(x)
        g2.launch(s.cuda_stream)
        s.synchronize()
        assert torch.equal(f, want)


# rows of 8 to 129 vectors around the 16, 32 and 64 lanes a run can take, whole
# and ending in a part of a vector; from the shortest rows that take runs
@pytest.mark.parametrize("dtype,inners", [("f64", (16, 17, 32, 33, 34, 63, 64, 65, 66, 127, 129, 131, 257)),
                                          ("f32", (32, 33, 63, 64, 65, 67, 68, 127, 129, 130, 255, 259, 513))])
@pytest.mark.parametrize("b", [None, 1, "inner"])
def test_short_and_unaligned_windows_bitwise_general_path(dtype, inners, b):
    """Rows shorter than a wavefront's slice (several runs per wavefront) and
    rows of a length that vectors do not divide, with and without b, give the
    general path's bits, also where N leaves the last run and the last group
    of runs short."""
    dt, tdt = (hb.F64, torch.float64) if dtype == "f64" else (hb.F32, torch.float32)
    for N, h in ((7, 1), (24, 2)):
        _, prog = hb.cs_program(N, h, hb.CS_LAGRANGE)
        for inner in inners:
            p = hb.cs_program(N, h, hb.CS_LAGRANGE)[1] if b else prog
            rng = np.random.default_rng(inner)
            if b:
                n = inner if b == "inner" else 1
                for f in (0, 3):
                    p.add_vector([(f, f + 1), (0, N), (-h, 0)], rng.normal(size=N * h * n), ninner=n)
            pw = hb.Plan(p, inner=inner, dtype=dt)
            pr = hb.Plan(p, inner=inner, dtype=dt, windows=False)
            assert any("k_apply_win" in k for k in pw.kernels())
            x = torch.from_numpy(rng.normal(size=(p.grid.cells, inner))).to(tdt).cuda()
            want, got = x.clone(), x.clone()
            hb.apply(pr, want)
            hb.apply(pw, got)
            torch.cuda.synchronize()
            assert torch.equal(got, want), (N, inner)


@pytest.mark.parametrize("dtype,inners", [("f64", (15, 16, 17, 33, 64, 66, 127, 129, 131)),
                                          ("f32", (31, 32, 33, 65, 129, 130, 255, 259))])
def test_batch_windows_bitwise_plain(dtype, inners):
    """A batch of plans whose rows take each form of the runs, with a plan with
    b and one built without windows among them, in shapes whose workgroups
    hold 1 to 4 items and loop over them."""
    dt, tdt = (hb.F64, torch.float64) if dtype == "f64" else (hb.F32, torch.float32)
    plans, inputs, want = [], [], []
    for k, inner in enumerate(inners):
        N, h = 9 + 4 * k, 1 + k % 3
        _, prog = hb.cs_program(N, h, hb.CS_LAGRANGE)
        if k == 2:
            prog.add_vector([(0, 1), (0, N), (-h, 0)], np.linspace(-1, 1, N * h))
        plans.append(hb.Plan(prog, inner=inner, dtype=dt, windows=k != 3))
        inputs.append(torch.from_numpy(np.random.default_rng(k).normal(size=(prog.grid.cells, inner))).to(tdt).cuda())
        want.append(inputs[-1].clone())
        hb.apply(plans[-1], want[-1])
    batch = hb.Batch(plans)
    for tune in (None, dict(block=64, persistent=0), dict(block=192, persistent=0), dict(block=256, persistent=50)):
        fields = [x.clone() for x in inputs]
        batch.bind(fields)
        if tune:
            batch.tune = {**batch.tune, **tune}
        batch.apply()
        torch.cuda.synchronize()
        assert all(torch.equal(f, w) for f, w in zip(fields, want)), tune


@pytest.mark.parametrize("rows,inner,dtype", [("lagrange", 33, "f64"), ("lagrange", 64, "f32"), ("quad", 3, "f64"),
                                              ("quad", 40, "f64")])
@pytest.mark.parametrize("ninner", [1, "inner"])
def test_corner_rows_with_b_ride_in_the_strips_launch(rows, inner, dtype, ninner):
    """b on zero rows (one corner of each face): the values are b, and the
    adjoint zeroes the rows."""
    dt, tdt = (hb.F64, torch.float64) if dtype == "f64" else (hb.F32, torch.float32)
    N, h = 11, 2
    n = inner if ninner == "inner" else 1
    p = hb.Program(hb.Grid.cubed_sphere(N, h))
    if rows == "quad":
        p.cs_add_quadrature(N, h, 2)
    else:
        p = hb.cs_program(N, h, hb.CS_LAGRANGE)[1]
    rng = np.random.default_rng(inner)
    b = rng.normal(size=(6, h * h, n))
    for f in range(6):
        p.add_vector([(f, f + 1), (-h, 0), (N, N + h)], b[f], ninner=n)
    plan = hb.Plan(p, inner=inner, dtype=dt)
    x = torch.from_numpy(rng.normal(size=(p.grid.cells, inner))).to(tdt).cuda()
    hb.apply(plan, x)
    W = N + 2 * h
    got = x.view(6, W, W, inner)[:, :h, N + h:].reshape(6, h * h, inner)
    want = torch.from_numpy(b).to(tdt).cuda().expand(6, h * h, inner) if n == 1 else torch.from_numpy(b).to(tdt).cuda()
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    hb.apply_adjoint(plan, x)
    torch.cuda.synchronize()
    assert (x.view(6, W, W, inner)[:, :h] == 0).all()


def one_strip_and_b(N, h, inner, ninner, rows):
    """A cubed sphere's ghosts: matrix rows on one side of face 0 (4 consecutive
    cells along the side, or their 4 x 4 square), b alone on every other side;
    and the expected values as (box, values or None for the matrix rows)."""
    p = hb.Program(hb.Grid.cubed_sphere(N, h))
    rng = np.random.default_rng(inner)
    W = N + 2 * h
    J, I = (a.ravel() for a in np.meshgrid(np.arange(N), np.arange(-h, 0), indexing="ij"))
    base = np.clip(J, 0, N - 4)
    near = 1 if rows == "ell" else 4
    cols = np.stack([(base + a + h) * W + (I + h if rows == "ell" else 0) + b + h
                     for a in range(4) for b in range(near)], 1)
    if rows == "ell":
        p.add_ell([(0, 1), (0, N), (-h, 0)], 4, cols, np.full(cols.shape, 0.25))
    else:
        p.add_csr([(0, 1), (0, N), (-h, 0)], np.arange(len(J) + 1) * 16, cols, np.full(cols.shape, 1 / 16))
    boxes = []
    for f in range(6):
        for box in ([(0, N), (-h, 0)], [(0, N), (N, N + h)], [(-h, 0), (0, N)], [(N, N + h), (0, N)]):
            if f or box != [(0, N), (-h, 0)]:
                v = rng.normal(size=(N * h, ninner))
                p.add_vector([(f, f + 1)] + box, v, ninner=ninner)
                boxes.append((f, box, v))
    return p, boxes, cols


# row vectors: whole and ending in a part, fewer and more than a workgroup's 256 threads
@pytest.mark.parametrize("inner,dtype,rows", [(16, "f64", "ell"), (33, "f64", "ell"), (32, "f32", "ell"),
                                              (137, "f32", "ell"), (1030, "f32", "ell"), (514, "f64", "ell"),
                                              (1, "f64", "quad"), (3, "f32", "quad"), (64, "f64", "quad")])
@pytest.mark.parametrize("scalar", [True, False])
def test_most_rows_b_only(inner, dtype, rows, scalar):
    dt, tdt = (hb.F64, torch.float64) if dtype == "f64" else (hb.F32, torch.float32)
    N, h = 13, 3
    p, boxes, cols = one_strip_and_b(N, h, inner, 1 if scalar else inner, rows)
    plan = hb.Plan(p, inner=inner, dtype=dt)
    x = torch.from_numpy(np.random.default_rng(1).integers(-8, 8, (p.grid.cells, inner))).to(tdt).cuda()
    want = x.clone()
    W = N + 2 * h
    w6 = want.view(6, W, W, inner)
    for f, (bj, bi), v in boxes:
        side = torch.from_numpy(v).to(tdt).cuda().view(bj[1] - bj[0], bi[1] - bi[0], -1)
        w6[f, bj[0] + h:bj[1] + h, bi[0] + h:bi[1] + h] = side
    strip = x[torch.from_numpy(cols).cuda()].double().mean(1).to(tdt)  # small whole numbers: exact
    w6[0, h:N + h, :h] = strip.view(N, h, inner)
    hb.apply(plan, x)
    torch.cuda.synchronize()
    assert torch.equal(x, want)


@pytest.mark.parametrize("N,inner", [(384, 32), (192, 137)])
def test_most_rows_b_only_cost_no_more_than_the_row_kernel(N, inner):
    """b-only rows that ride in the window launch take about the row kernel's
    time (one value per lane took 1.5 to 2 times as long)."""
    p, _, _ = one_strip_and_b(N, 3, inner, 1, "ell")
    s = torch.cuda.Stream()
    ms = []
    for windows in (True, False):
        plan = hb.Plan(p, inner=inner, dtype=hb.F32, windows=windows)
        fields = [torch.zeros(plan.nelem, device="cuda") for _ in range(2)]
        ms.append(min(hb.time_apply(plan, fields, 40, s.cuda_stream) for _ in range(9)))
    assert ms[0] <= 1.25 * ms[1]
