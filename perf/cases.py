"""Cases that time this library's public entry points as a program that uses it would call them.

A case is a dict of plain values; ``op`` names the call and the other keys the grid, the rows of the boundary
condition, the field's layout and its type:

* ``apply``: one ``apply`` of a cubed-sphere program (``rows``: ``sync`` rotated copies, ``lagrange`` 4-point
  interpolation, ``quad`` cell averages by quadrature with 16-25 entries a row, ``average`` copies plus the mean of the
  co-located points of a vertex-centred grid);
* ``graph``: the applies of the stages of one time step, captured once and replayed;
* ``adjoint``: one ``apply_adjoint`` on a field of output gradients;
* ``batch``: one batched apply over grids of different sizes;
* ``stencil27``: the 27-point operator on Cartesian blocks with its halo exchange, fused or as two calls;
* ``consumer``: the radius-1 cross stencil reading the boundary condition's ghosts, fused or as two calls.
"""
import functools
import math
import random

import numpy as np
import torch

import paper_2605_14780_amd as hb

TYPES = {"f64": (hb.F64, torch.float64, 8), "f32": (hb.F32, torch.float32, 4)}
CROSS = ([(0, 0, 0), (0, 0, 1), (0, 0, -1), (0, 1, 0), (0, -1, 0)], [-4.0, 1.0, 1.0, 1.0, 1.0])
BATCH_SIZES = (48, 96, 192, 384, 768)
LARGEST_FIELD = 1.5e9  # bytes of a drawn field: below the largest listed one


def listed():
    cs = {"h": 3, "dtype": "f64", "order": "point", "vector": True, "b": False}
    return [
        # the smallest call: one variable on one level of a coarse sphere, where launching is what costs
        {**cs, "name": "c48_sync", "op": "apply", "rows": "sync", "N": 48, "inner": 1, "vector": False},
        # shallow water (h, u, v): the four stage fields of one Runge-Kutta step, replayed as a graph every step
        {**cs, "name": "c90_shallow_water_step", "op": "graph", "rows": "quad", "N": 90, "inner": 3, "stages": 4},
        # an atmosphere model's full state: 64 levels of h, a tracer and (u, v)
        {**cs, "name": "c384_state", "op": "apply", "rows": "lagrange", "N": 384, "inner": 256},
        # one single-precision tracer on an odd number of levels, with an affine part
        {**cs, "name": "c384_tracer_f32", "op": "apply", "rows": "lagrange", "N": 384, "inner": 137, "dtype": "f32",
         "vector": False, "b": True},
        # the same state with high-order ghost averages: wide rows
        {**cs, "name": "c384_state_quadrature", "op": "apply", "rows": "quad", "N": 384, "inner": 256},
        # the same state kept level by level, as most models store it
        {**cs, "name": "c384_state_planes", "op": "apply", "rows": "lagrange", "N": 384, "inner": 256,
         "order": "plane"},
        # a finer grid's gradients: 8 levels of h, a tracer and (u, v)
        {**cs, "name": "c768_adjoint", "op": "adjoint", "rows": "lagrange", "N": 768, "h": 2, "inner": 32},
        # gradients through the wide rows
        {**cs, "name": "c192_quadrature_adjoint", "op": "adjoint", "rows": "quad", "N": 192, "inner": 64},
        # an ensemble of single-precision grids of different sizes and level counts
        {"name": "batch_24_grids", "op": "batch", "grids": 24, "draw": 4, "dtype": "f32"},
        # HPCG's operator on 2 x 2 x 2 blocks of 128^3 with its halo exchange
        {"name": "hpcg_256", "op": "stencil27", "blocks": 2, "n": 128, "periodic": False, "fused": True,
         "dtype": "f64"},
        # a horizontal diffusion of the full state: the largest pass
        {**cs, "name": "c384_state_diffusion", "op": "consumer", "rows": "lagrange", "N": 384, "h": 1, "inner": 256,
         "fused": True},
        # a vertex-centred grid: ghosts and the averages of the points that faces share
        {**cs, "name": "c385_edge_average", "op": "apply", "rows": "average", "N": 385, "inner": 256,
         "vector": False},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op, rows = rng.choice([("apply", "sync"), ("apply", "lagrange"), ("apply", "lagrange"), ("apply", "quad"),
                           ("apply", "quad"), ("apply", "average"), ("graph", "quad"), ("graph", "lagrange"),
                           ("adjoint", "lagrange"), ("adjoint", "quad"), ("batch", ""), ("stencil27", ""),
                           ("consumer", "lagrange")])
    dtype = rng.choice(["f64", "f64", "f32"])
    if op == "batch":
        return {"op": op, "grids": rng.randint(4, 24), "draw": rng.randint(100, 10 ** 6), "dtype": dtype}
    if op == "stencil27":
        return {"op": op, "blocks": rng.randint(1, 2), "n": rng.randint(24, 128), "periodic": rng.random() < 0.5,
                "fused": rng.random() < 0.7, "dtype": dtype}
    small = op == "graph"
    case = {"op": op, "rows": rows, "N": _log_int(rng, 48, 128 if small else 512 if rows == "quad" else 768),
            "h": 1 if op == "consumer" else rng.randint(1, 4), "dtype": dtype, "order": "point",
            "vector": False, "b": False}
    room = LARGEST_FIELD / (6 * (case["N"] + 2 * case["h"]) ** 2 * TYPES[dtype][2])
    inner = _log_int(rng, 1, max(1, min(8 if small else 256, int(room))))
    if rows != "average" and rng.random() < 0.5 and inner >= 3:
        inner = 4 * max(1, inner // 4) if inner >= 8 else 3
        case["vector"] = True
    case["inner"] = inner
    if small:
        case["stages"] = rng.randint(2, 4)
    elif op == "consumer":
        case["fused"] = rng.random() < 0.5
    elif op == "apply" and rows == "lagrange":
        case["b"] = rng.random() < 0.25
        case["order"] = rng.choice(["point", "plane"])
    return case


# ---- the geometry of the rows, from 3-D positions ------------------------------------------
FRAMES = np.array([[[1, 0, 0], [0, 1, 0], [0, 0, 1]], [[0, 1, 0], [-1, 0, 0], [0, 0, 1]],
                   [[-1, 0, 0], [0, -1, 0], [0, 0, 1]], [[0, -1, 0], [1, 0, 0], [0, 0, 1]],
                   [[0, 0, 1], [0, 1, 0], [-1, 0, 0]], [[0, 0, -1], [0, 1, 0], [1, 0, 0]]], dtype=np.float64)


def _layout(case):
    """(lo, stride, len) of the two vector components among a cell's values, or None."""
    if not case["vector"]:
        return None
    n = case["inner"]
    return (1, 1, 1) if n == 3 else (n // 2, n // 4, n // 4)


def _neighbour(f, normal):
    return int(np.argmax(FRAMES[:, 0] @ normal))


def _index(P, g, N):
    """Fractional (j, i) of the rays through P on face g."""
    c, e1, e2 = FRAMES[g]
    D = math.pi / (2 * N)
    return tuple((np.arctan((P @ e) / (P @ c)) + math.pi / 4) / D - 0.5 for e in (e2, e1))


def _lagrange(s, N):
    base = np.clip(np.floor(s).astype(np.int64) - 1, 0, N - 4)
    d = [s - (base + m) for m in range(4)]
    return base, [-d[1] * d[2] * d[3] / 6, d[0] * d[2] * d[3] / 2, -d[0] * d[1] * d[3] / 2, d[0] * d[1] * d[2] / 6]


@functools.lru_cache(maxsize=4)
def _sides(N, h, rows):
    """Per face side: (ghost cells, source cells, weights, rotation of (u, v)); sources and weights by row and entry."""
    W, D = N + 2 * h, math.pi / (2 * N)
    cell = lambda f, j, i: (f * W + j + h) * W + i + h  # noqa: E731
    t, k = np.meshgrid(np.arange(N), np.arange(h), indexing="ij")
    t, k = t.ravel(), k.ravel()
    out = []
    for f in range(6):
        c, e1, e2 = FRAMES[f]
        for axis in (0, 1):  # ghosts beyond an end of i, then of j
            for high in (False, True):
                across = N + k if high else -1 - k
                j, i = (t, across) if axis == 0 else (across, t)
                n, e = ((e1, e2) if axis == 0 else (e2, e1))
                normal = n if high else -n
                g = _neighbour(f, normal)
                at = lambda v: np.tan(-math.pi / 4 + (v + 0.5) * D)[..., None]  # noqa: E731
                if rows == "quad":
                    x, wx = np.polynomial.legendre.leggauss(2)
                    cols, wts = [], []
                    for xb, wb in zip(x / 2, wx / 2):
                        for xa, wa in zip(x / 2, wx / 2):
                            sj, si = _index(c + at(i + xa) * e1 + at(j + xb) * e2, g, N)
                            bj, wj = _lagrange(sj, N)
                            bi, wi = _lagrange(si, N)
                            cols += [cell(g, bj + a, bi + b) for a in range(4) for b in range(4)]
                            wts += [wa * wb * wj[a] * wi[b] for a in range(4) for b in range(4)]
                    cols, wts = np.stack(cols, 1), np.stack(wts, 1)
                else:
                    sj, si = _index(c + at(i) * e1 + at(j) * e2, g, N)
                    # the neighbour's grid line through the ghost lies k lines from the shared edge
                    ti, tj = _index((c + normal + at(t) * e), g, N)[::-1]
                    lines_i = np.abs(ti - np.round(ti)).max() > 0.25  # i is constant (-1/2 or N - 1/2) on the edge
                    edge, s, along = (ti, sj, tj) if lines_i else (tj, si, ti)
                    line = np.where(edge > N / 2, N - 1 - k, k)
                    node = lambda v: cell(g, v, line) if lines_i else cell(g, line, v)  # noqa: E731
                    if rows == "lagrange":
                        base, w = _lagrange(np.where(np.abs(s - np.round(s)) <= 1e-9, np.round(s), s), N)
                        cols, wts = np.stack([node(base + m) for m in range(4)], 1), np.stack(w, 1)
                    else:
                        cols = node(np.round(along).astype(np.int64))[:, None]
                        wts = np.ones(cols.shape)
                out.append((cell(f, j, i), cols, wts, _rotation(f, normal, g)))
    return out


def _rotation(f, normal, g):
    """(u, v) of a ghost of face f beyond `normal` from those of its neighbour g: tangents at the edge's midpoint."""
    Q = FRAMES[f, 0] + normal

    def tangents(face):
        c, e1, e2 = FRAMES[face]
        p = Q / (Q @ c)
        v = [e - p * (p @ e) / (p @ p) for e in (e1, e2)]
        return np.stack([x / np.linalg.norm(x) for x in v])

    return np.rint(tangents(f) @ tangents(g).T).astype(int)


@functools.lru_cache(maxsize=4)
def _shared_points(N, h):
    """Cells of a vertex-centred grid's face boundaries, and the number of the 3-D point each lies on."""
    W, t = N + 2 * h, np.tan(-math.pi / 4 + np.arange(N) * math.pi / (2 * (N - 1)))
    f, j, i = np.meshgrid(np.arange(6), np.arange(N), np.arange(N), indexing="ij")
    on = ((j % (N - 1) == 0) | (i % (N - 1) == 0))
    f, j, i = f[on], j[on], i[on]
    p = FRAMES[f, 0] + t[i][:, None] * FRAMES[f, 1] + t[j][:, None] * FRAMES[f, 2]
    p /= np.linalg.norm(p, axis=1, keepdims=True)
    point = np.unique(np.round(p * 1e7).astype(np.int64) + 0, axis=0, return_inverse=True)[1].reshape(-1)
    return (f * W + j + h) * W + i + h, point


def _batch_grids(case):
    rng = random.Random(case["draw"])
    return [(rng.choice(BATCH_SIZES), rng.randint(2, 4), rng.randint(1, 128)) for _ in range(case["grids"])]


# ---- inputs ---------------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _sphere_field(N, h, inner, dtype, gen, order="point"):
    """Smooth functions of the position, one per value of a cell, with a little noise; stale values in the ghosts."""
    W, dev = N + 2 * h, "cuda"
    t = torch.tan(-math.pi / 4 + (torch.arange(-h, N + h, device=dev) + 0.5) * (math.pi / (2 * N))).to(dtype)
    fr = torch.tensor(FRAMES, device=dev, dtype=dtype)
    p = fr[:, None, None, 0] + t[None, None, :, None] * fr[:, None, None, 1] + t[None, :, None, None] * fr[:, None, None, 2]
    p = (p / p.norm(dim=-1, keepdim=True)).reshape(-1, 3)
    x, y, z = p.unbind(1)
    basis = torch.stack([torch.ones_like(x), x, y, z, x * y, y * z, z * x, x * x - y * y, 3 * z * z - 1], 1)
    coef = torch.randn(9, inner, device=dev, dtype=dtype, generator=gen)
    if order == "plane":
        return torch.randn(inner, 6 * W * W, device=dev, dtype=dtype, generator=gen).mul_(1e-3).addmm_(coef.t(), basis.t())
    return torch.randn(6 * W * W, inner, device=dev, dtype=dtype, generator=gen).mul_(1e-3).addmm_(basis, coef)


def _gradient(case, gen):
    W = case["N"] + 2 * case["h"]
    return torch.randn(6 * W * W, case["inner"], device="cuda", dtype=TYPES[case["dtype"]][1], generator=gen)


def _blocks(case, seed):
    """The Cartesian field, block by block with a one-cell halo of stale values."""
    nb, n, dtype = case["blocks"], case["n"], TYPES[case["dtype"]][1]
    return torch.rand(nb ** 3, n + 2, n + 2, n + 2, device="cuda", dtype=dtype, generator=_generator(seed)) * 2 - 1


def _b_values(case, seed):
    """One value per ghost row of each face side (rows by the last coordinate fastest)."""
    g, n = _generator(seed + 7), case["N"] * case["h"]
    return [torch.randn(n, device="cuda", dtype=torch.float64, generator=g).mul_(0.1) for _ in range(24)]


def _side_boxes(N, h):
    return [[(f, f + 1)] + b for f in range(6) for b in
            ([(0, N), (-h, 0)], [(0, N), (N, N + h)], [(-h, 0), (0, N)], [(N, N + h), (0, N)])]


def _cs_program(case):
    N, h, rows = case["N"], case["h"], case["rows"]
    if rows == "lagrange":
        return hb.cs_program(N, h, hb.CS_LAGRANGE, vector=case["vector"])[1]
    prog = hb.Program(hb.Grid.cubed_sphere(N, h))
    if rows == "quad":
        prog.cs_add_quadrature(N, h, 2, vector=case["vector"])
    else:
        prog.cs_add(N, h, hb.CS_SYNC, vector=case["vector"])
        if rows == "average":
            prog.cs_add_edge_average(N)
    return prog


def prepare(case, seed):
    op, (hd, td, _) = case["op"], TYPES[case["dtype"]]
    if op == "batch":
        plans, fields, gen = [], [], _generator(seed)
        for N, h, levels in _batch_grids(case):
            plans.append(hb.Plan(hb.cs_program(N, h, hb.CS_LAGRANGE)[1], inner=levels, dtype=hd))
            fields.append(_sphere_field(N, h, levels, td, gen))
        batch = hb.Batch(plans)
        batch.bind(fields)
        return {"op": op, "batch": batch, "fields": fields}
    if op == "stencil27":
        nb, n = [case["blocks"]] * 3, [case["n"]] * 3
        prog = hb.Program(hb.Grid.cartesian(nb, n, 1))
        prog.cart_add_halo(nb, n, 1, 7 if case["periodic"] else 0)
        y = torch.empty(case["blocks"] ** 3 * case["n"] ** 3, device="cuda", dtype=td)
        return {"op": op, "plan": hb.Plan(prog, inner=1, dtype=hd), "x": _blocks(case, seed), "y": y, "fused": case["fused"]}
    prog, gen = _cs_program(case), _generator(seed)
    if case["b"]:
        for box, values in zip(_side_boxes(case["N"], case["h"]), _b_values(case, seed)):
            prog.add_vector(box, values.cpu().numpy())
    plan = hb.Plan(prog, inner=case["inner"], vec=_layout(case), dtype=hd,
                   order=hb.PLANE_MAJOR if case["order"] == "plane" else hb.POINT_MAJOR)
    field = lambda: _sphere_field(case["N"], case["h"], case["inner"], td, gen, case["order"])  # noqa: E731
    state = {"op": op, "plan": plan}
    if op == "adjoint":
        plan.kernels(hb.OP_ADJOINT)  # builds the transposed tables, once per plan
        state["x"] = _gradient(case, gen)
    elif op == "graph":
        state["x"] = [field() for _ in range(case["stages"])]
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        state["graph"] = hb.ApplyGraph(plan, state["x"], case["stages"], stream=stream.cuda_stream)
        torch.cuda.current_stream().wait_stream(stream)
    else:
        state["x"] = field()
        if op == "consumer":
            state["consumer"] = hb.Consumer(plan, *CROSS)
            state["y"] = torch.empty(6 * case["N"] ** 2, case["inner"], device="cuda", dtype=td)
            state["fused"] = case["fused"]
    return state


def run(state):
    op = state["op"]
    if op == "apply":
        return hb.apply(state["plan"], state["x"])
    if op == "graph":
        state["graph"].launch()
        return state["x"]
    if op == "adjoint":
        return hb.apply_adjoint(state["plan"], state["x"])
    if op == "batch":
        state["batch"].apply()
        return state["fields"]
    if op == "stencil27":
        if state["fused"]:
            hb.fused_stencil27(state["plan"], state["x"], state["y"])
        else:
            hb.apply(state["plan"], state["x"])
            hb.stencil27(state["plan"], state["x"], state["y"])
        return [state["x"], state["y"]]
    if state["fused"]:
        return state["consumer"].apply(state["x"], state["y"], fused=True)
    hb.apply(state["plan"], state["x"])
    return [state["x"], state["consumer"].apply(state["x"], state["y"], fused=False)]


# ---- what a pass cannot do without ------------------------------------------------------------
def _rows_work(N, h, rows, inner, size):
    """Values written and read once, and operations, of the ghost rows of one field."""
    sides = _sides(N, h, "sync" if rows == "average" else rows)
    source = np.unique(np.concatenate([s[1].ravel() for s in sides])).size
    ghost = 24 * N * h + 24 * h * h
    entries = {"lagrange": 4, "quad": 22}.get(rows, 1)
    return (ghost + source) * inner * size, 2 * entries * 24 * N * h * inner, ghost, source


def work(case):
    op, size = case["op"], TYPES[case["dtype"]][2]
    if op == "batch":
        each = [_rows_work(N, h, "lagrange", levels, size)[:2] for N, h, levels in _batch_grids(case)]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    if op == "stencil27":
        nb, n = case["blocks"], case["n"]
        ghosts = (n + 2) ** 3 - n ** 3
        return {"bytes": nb ** 3 * (2 * n ** 3 + ghosts) * size, "flops": nb ** 3 * n ** 3 * 28}
    N, inner = case["N"], case["inner"]
    nbytes, flops, ghost, source = _rows_work(N, case["h"], case["rows"], inner, size)
    if op == "graph":
        return {"bytes": nbytes * case["stages"], "flops": flops * case["stages"]}
    if op == "adjoint":  # gradients of the ghosts read and zeroed, those of the sources read and written
        return {"bytes": 2 * nbytes, "flops": flops}
    if op == "consumer":
        stencil = 2 * 6 * N * N * inner * size
        return {"bytes": stencil + (0 if case["fused"] else ghost * inner * size), "flops": flops + 10 * 6 * N * N * inner}
    if case["rows"] == "average":
        shared = _shared_points(N, case["h"])[0].size
        return {"bytes": nbytes + shared * inner * size, "flops": flops + 4 * shared * inner}
    return {"bytes": nbytes, "flops": flops}


# ---- the same results in 64 bits, in plain torch ------------------------------------------------
def _rotate(y, R, vec, transpose=False):
    if vec is not None:
        lo, stride, n = vec
        R = R.T if transpose else R
        u, v = y[:, lo:lo + n].clone(), y[:, lo + stride:lo + stride + n].clone()
        y[:, lo:lo + n] = int(R[0, 0]) * u + int(R[0, 1]) * v
        y[:, lo + stride:lo + stride + n] = int(R[1, 0]) * u + int(R[1, 1]) * v
    return y


def _on_gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _zero_corners(x, N, h):
    v = x.view(6, N + 2 * h, N + 2 * h, -1)
    for a in (slice(0, h), slice(N + h, None)):
        for b in (slice(0, h), slice(N + h, None)):
            v[:, a, b] = 0


def _exact_apply(x, N, h, rows, vec=None, b=None):
    out = x.clone()
    _zero_corners(out, N, h)
    for n, (dst, cols, w, R) in enumerate(_sides(N, h, rows)):
        cols, w = _on_gpu(cols), _on_gpu(w)
        y = torch.zeros(len(dst), x.shape[1], device="cuda", dtype=torch.float64)
        for m in range(cols.shape[1]):
            y += w[:, m, None] * x[cols[:, m]]
        y = _rotate(y, R, vec)
        if b is not None:  # b goes by the box's rows; these rows go by the tangential index first
            t = b[n].view(N, h) if n % 4 < 2 else b[n].view(h, N).t()
            layers = t if n % 2 else t.flip(1)  # the box counts layers upwards, these rows away from the face
            y += layers.reshape(-1, 1)
        out[_on_gpu(dst)] = y
    return out


def _exact_adjoint(g, N, h, rows, vec):
    out = g.clone()
    for dst, cols, w, R in _sides(N, h, rows):
        dst, cols, w = _on_gpu(dst), _on_gpu(cols), _on_gpu(w)
        y = _rotate(g[dst], R, vec, transpose=True)
        out[dst] = 0
        for m in range(cols.shape[1]):
            out.index_add_(0, cols[:, m], w[:, m, None] * y)
    _zero_corners(out, N, h)
    return out


def _exact_blocks(case, seed):
    nb, n = case["blocks"], case["n"]
    x = _blocks(case, seed).double()
    inner = x[:, 1:-1, 1:-1, 1:-1].view(nb, nb, nb, n, n, n).permute(0, 3, 1, 4, 2, 5).reshape(1, 1, nb * n, nb * n, nb * n)
    pad = torch.nn.functional.pad(inner, [1] * 6, mode="circular" if case["periodic"] else "constant")[0, 0]
    total = torch.zeros_like(inner[0, 0])
    for dz in range(3):
        for dy in range(3):
            for dx in range(3):
                total += pad[dz:dz + nb * n, dy:dy + nb * n, dx:dx + nb * n]
    y = (27 * inner[0, 0] - total).view(nb, n, nb, n, nb, n).permute(0, 2, 4, 1, 3, 5).reshape(-1)
    x = torch.stack([pad[z * n:z * n + n + 2, a * n:a * n + n + 2, c * n:c * n + n + 2]
                     for z in range(nb) for a in range(nb) for c in range(nb)])
    return [x, y]


def exact(case, seed):
    op, td = case["op"], TYPES[case["dtype"]][1]
    if op == "stencil27":
        return _exact_blocks(case, seed)
    gen = _generator(seed)
    if op == "batch":
        return [_exact_apply(_sphere_field(N, h, levels, td, gen).double(), N, h, "lagrange")
                for N, h, levels in _batch_grids(case)]
    N, h, rows, vec = case["N"], case["h"], case["rows"], _layout(case)
    if op == "adjoint":
        return _exact_adjoint(_gradient(case, gen).double(), N, h, rows, vec)
    fields = [_sphere_field(N, h, case["inner"], td, gen, case["order"]).double() for _ in range(case.get("stages", 1))]
    if case["order"] == "plane":
        fields = [x.t().contiguous() for x in fields]
    if rows == "average":
        x = fields[0]
        out = _exact_apply(x, N, h, "sync")
        cells, point = (_on_gpu(a) for a in _shared_points(N, h))
        count = torch.bincount(point).double()[:, None]
        mean = torch.zeros(count.shape[0], x.shape[1], device="cuda", dtype=torch.float64).index_add_(0, point, x[cells]) / count
        out[cells] = mean[point]
        return out
    b = [v.to(td).double() for v in _b_values(case, seed)] if case["b"] else None
    outs = [_exact_apply(x, N, h, rows, vec, b) for x in fields]
    if op == "graph":
        return outs
    if op == "consumer":
        x, W = outs[0], N + 2 * h
        v = x.view(6, W, W, -1)
        y = 0
        for (_, dj, di), w in zip(*CROSS):
            y = y + w * v[:, h + dj:h + dj + N, h + di:h + di + N]
        y = y.reshape(6 * N * N, -1)
        return y if case["fused"] else [x, y]
    return outs[0].t().contiguous() if case["order"] == "plane" else outs[0]
