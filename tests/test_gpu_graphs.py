"""Graphs of applies beside what else a program captures."""
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
