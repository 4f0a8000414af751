"""The adjoint kernels at the ends of their ranges."""
import numpy as np
import pytest

from helpers import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch

    import paper_2605_14780_amd as hb


@pytest.mark.parametrize("inner,nzero", [(1 << 25 | 1, 65), (3, 130), (600, 70)])
def test_unread_ghost_rows_are_zeroed(inner, nzero):
    """Covered ghosts that no source reads, more than one workgroup's 64 of
    them: rows of so many single values that 64 of them pass 2^31, rows of
    fewer and of more vectors than a workgroup has threads."""
    n = nzero + 3
    g = hb.Grid([0], [n])
    g.add_block([(0, n)], [(n - 2, n)])
    p = hb.Program(g)
    p.add_zero([(0, nzero)])
    p.add_csr([(nzero, nzero + 1)], [0, 9], [n - 2] * 9, [0.5] * 9)  # more entries than the fixed-width tables hold
    plan = hb.Plan(p, inner=inner, dtype=hb.F32)
    assert any("k_adjoint_wide" in k for k in plan.kernels(hb.OP_ADJOINT))
    x = torch.ones(n, inner, device="cuda")
    hb.apply_adjoint(plan, x)
    torch.cuda.synchronize()
    want = [0.0] * (nzero + 1) + [5.5, 1.0]
    assert [float(r.min()) for r in x] == want and [float(r.max()) for r in x] == want
