"""Right-hand-side adjoint of a state with 2^26 lines of two cells (8192 x 8192 x 2,
27 GB for all arrays), where a wave per line makes 2^32 threads: more than a
launch holds along one axis. The state and cotangent repeat a 64 x 64 x 2 periodic
domain, so the result must repeat that domain's.

The small domain's cells at its periodic edges gather the same contributions in
another order: within 1e-5 of each field's maximum, as for every change of order
in single precision.
"""
import pytest
import torch

import paper_1901_02955_amd as snap
import workloads as wl

pytestmark = pytest.mark.gpu


def adjoint(grid, inner, rb):
    dg = snap.device_grid(grid, dtype=inner.dtype)
    q = torch.empty(dg.shape, dtype=inner.dtype, device="cuda")
    rbar = torch.empty(dg.interior_shape, dtype=inner.dtype, device="cuda")
    n, m = inner.shape[2], inner.shape[3]
    view = grid.interior(q)
    for j in range(0, grid.ny, n):
        for i in range(0, grid.nx, m):
            view[:, :, j:j + n, i:i + m] = inner
            rbar[:, :, j:j + n, i:i + m] = rb
    out = torch.empty_like(rbar)
    snap.snap_rhs_adjoint(dg, q, rbar, out, snap.workspace(dg, snap.SNAP_OP_RHS_ADJ))
    return out


def test_many_short_lines():
    n = 64
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 35e9:
        pytest.skip("needs 35 GB of free device memory")
    grid, _ = wl.dry_grid(n, n, 2, 200.0 * n, 200.0 * n, 300.0, bc=(0, 0, 1))
    inner = torch.as_tensor(grid.interior(wl.random_smooth_state(grid, 5)).copy()).float().cuda()
    rb = torch.as_tensor(wl.seeded_normal(grid.interior_shape, 6)).float().cuda()
    ref = adjoint(grid, inner, rb)
    k = 8192
    # blocks of many periods at a time: the same state, written in few copies
    big = grid.copy(nx=k, ny=k)
    wide = inner.repeat(1, 1, k // n // 2, k // n // 2)
    print(f"[many lines] {k} x {k} x 2", flush=True)
    out = adjoint(big, wide, rb.repeat(1, 1, k // n // 2, k // n // 2))
    for v in range(grid.nvar):
        tiles = out[v].reshape(2, k // n, n, k // n, n)
        err = (tiles - ref[v][:, None, :, None, :]).abs().max()
        assert err <= 1e-5 * ref[v].abs().max(), (v, float(err))
    del out, wide, tiles
    torch.cuda.empty_cache()
