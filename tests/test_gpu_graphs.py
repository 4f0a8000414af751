"""Graphs of applies beside what else a program captures."""
import time

import pytest

from helpers import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch

    import paper_2605_14780_amd as hb


@pytest.mark.parametrize("nfields,reps", [(1, 1), (2, 2), (3, 9), (11, 20)])
def test_graph_made_and_dropped_while_another_stream_captures(nfields, reps):
    """A capture that the program has open takes no notice of a graph that is
    created, or destroyed, on another stream: both replay as they should."""
    p = hb.Program(hb.Grid.cubed_sphere(10, 2))
    p.cs_add(10, 2, hb.CS_SYNC)
    plan = hb.Plan(p, inner=2)
    gen = torch.Generator("cuda").manual_seed(nfields)
    start = [torch.randn(plan.nelem, device="cuda", dtype=torch.float64, generator=gen) for _ in range(nfields)]
    want = [hb.apply(plan, x.clone()) if k < reps else x.clone() for k, x in enumerate(start)]
    xs = [x.clone() for x in start]
    y = torch.zeros(64, device="cuda")
    s = torch.cuda.Stream()
    kept = hb.ApplyGraph(plan, xs, reps, stream=s.cuda_stream)
    torch.cuda.synchronize()
    outer = torch.cuda.CUDAGraph()
    with torch.cuda.graph(outer):
        y.add_(1)
        made = hb.ApplyGraph(plan, xs, reps, stream=s.cuda_stream)
        del kept
        y.add_(1)
    for rep in range(3):
        for x, x0 in zip(xs, start):
            x.copy_(x0)
        y.zero_()
        outer.replay()
        torch.cuda.synchronize()
        made.launch(s.cuda_stream)
        torch.cuda.synchronize()
        assert (y == 2).all(), rep
        assert all(torch.equal(x, w) for x, w in zip(xs, want)), rep


@pytest.mark.parametrize("call", ["apply", "graph"])
def test_host_time_of_a_call_does_not_grow_with_the_tiles(call):
    """A call reads nothing per tile on the host: 27000 tiles cost it what 50
    do (a scan of them takes 12 us, a launch 3)."""
    host = {}
    for N, rows in ((384, 1), (8, 512)):
        p = hb.Program(hb.Grid.cubed_sphere(N, 3))
        p.cs_add(N, 3, hb.CS_SYNC)
        plan = hb.Plan(p, inner=1)
        plan.tune = {**plan.tune, "block": 64, "lanes_per_row": 1, "rows_per_tile": rows}
        x = torch.zeros(plan.nelem, device="cuda", dtype=torch.float64)
        s = torch.cuda.Stream()
        graph = hb.ApplyGraph(plan, [x], 1, stream=s.cuda_stream)
        once = (lambda: graph.launch(s.cuda_stream)) if call == "graph" else (lambda: hb.apply(plan, x, s.cuda_stream))
        times = []
        for _ in range(30):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(20):
                once()
            times.append((time.perf_counter() - t) / 20)
        host[plan.stats()["tiles"]] = min(times)
    (few, least), (many, most) = sorted(host.items())
    assert few < 60 and many > 27000
    assert most <= least + 8e-6
