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


def copies(n, inner, dtype, fan=1):
    """Ghost k of n copies cell k // fan of a 1-D block."""
    g = hb.Grid([0], [2 * n])
    g.add_block([(0, 2 * n)], [(n, 2 * n)])
    p = hb.Program(g)
    p.add_csr([(0, n)], np.arange(n + 1), n + np.arange(n) // fan, np.ones(n))
    return hb.Plan(p, inner=inner, dtype=dtype)


# the row lengths at which plans of few entries per source take another kernel:
# 128 bytes, 3 KiB where most sources have one entry, 8 KiB
@pytest.mark.parametrize("inner,fan,wide", [(15, 1, False), (16, 1, True), (384, 1, True), (385, 1, False),
                                            (1024, 4, True), (1026, 4, False), (4097, 4, False)])
def test_rows_of_every_length_take_a_kernel_and_sum_right(inner, fan, wide):
    """Small whole numbers: every order of a sum gives the same value."""
    n = 70
    plan = copies(n, inner, hb.F64, fan)
    assert any("k_adjoint_wide" in k for k in plan.kernels(hb.OP_ADJOINT)) == wide
    x = torch.randint(-9, 9, (2 * n, inner), device="cuda", generator=torch.Generator("cuda").manual_seed(inner)).double()
    want = x.clone()
    want[:n] = 0
    want.index_add_(0, n + torch.arange(n, device="cuda") // fan, x[:n])
    for call in (hb.apply_adjoint, hb.apply_adjoint_noalloc):
        got = x.clone()
        call(plan, got)
        torch.cuda.synchronize()
        assert torch.equal(got, want)


@pytest.mark.parametrize("inner,dtype", [(5, "f64"), (32, "f32"), (301, "f64")])
def test_source_of_more_ghosts_than_a_tile_stages(inner, dtype):
    """One cell that 300 ghosts read: the plan goes by the walking kernel,
    point-major, with and without allocation."""
    n, tdt = 300, torch.float64 if dtype == "f64" else torch.float32
    plan = copies(n, inner, hb.F64 if dtype == "f64" else hb.F32, fan=n)
    assert any("k_adjoint<" in k for k in plan.kernels(hb.OP_ADJOINT))
    x = torch.randint(-9, 9, (2 * n, inner), device="cuda", generator=torch.Generator("cuda").manual_seed(1)).to(tdt)
    want = x.clone()
    want[:n] = 0
    want[n] += x[:n].sum(0)
    for call in (hb.apply_adjoint, hb.apply_adjoint_noalloc):
        got = x.clone()
        call(plan, got)
        torch.cuda.synchronize()
        assert torch.equal(got, want)


# reader counters (shared rows x slices of 16 values) beyond the static array's
# 2^20: sources of 16 entries in long rows (the walking kernel's), of 8 in many
# rows (the LDS kernel's)
@pytest.mark.parametrize("n,entries,inner", [(200, 16, 100001), (16000, 2, 1279)])
def test_noalloc_without_room_for_the_counters(n, entries, inner):
    """The allocation-free call takes another kernel, with the same bits, on
    repeated calls too."""
    g = hb.Grid([0], [2 * n])
    g.add_block([(0, 2 * n)], [(n, 2 * n)])
    p = hb.Program(g)
    k, m = np.arange(n)[:, None], n // 4
    if entries == 2:  # four times as many ghosts as sources: nearly every ghost has sources of two tiles
        cols = np.hstack([k % m, (k * 4801 + k // m * 17) % m])
    else:
        cols = (k + np.arange(entries) * (n // entries)) % n
    p.add_csr([(0, n)], np.arange(n + 1) * entries, n + cols, np.ones((n, entries)))
    plan = hb.Plan(p, inner=inner, dtype=hb.F32)
    assert any("k_adjoint_wide" in k for k in plan.kernels(hb.OP_ADJOINT))
    gen = torch.Generator("cuda").manual_seed(n)
    x = torch.randint(-9, 9, (2 * n, inner), device="cuda", generator=gen, dtype=torch.int32).float()
    want = x.clone()  # small whole numbers: exact in any order
    want[:n] = 0
    for c in cols.T:
        want[n:].index_add_(0, torch.from_numpy(c).cuda(), x[:n])
    for call in (hb.apply_adjoint, hb.apply_adjoint_noalloc, hb.apply_adjoint_noalloc, hb.apply_adjoint):
        got = x.clone()
        call(plan, got)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
