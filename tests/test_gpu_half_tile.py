"""Right-hand side and step of the double-precision kernels with two to four tracers,
which have a half tile (16 x 8) beside the square one: both against the oracle on
grids of ragged tiles (one column, one row, less than a tile, exact multiples), and
the choice between them on sizes on either side of the rule.

Tolerances as for every double-precision right-hand side and step: 1e-12 of each
field's maximum.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_02955_amd as snap
import workloads as wl

pytestmark = pytest.mark.gpu


def case(size, nt, riemann):
    nx, ny, nz = size
    grid, _ = wl.dry_grid(nx, ny, nz, 200.0 * nx, 200.0 * ny, 150.0 * nz, bc=(nx % 2, 0, 1))
    grid.ntracer, grid.riemann = nt, riemann
    return grid, wl.random_smooth_state(grid, 40 + nt)


def rhs(grid, q):
    dg = snap.device_grid(grid)
    out = torch.empty(dg.interior_shape, dtype=torch.float64, device="cuda")
    snap.snap_rhs(dg, torch.as_tensor(q).cuda(), out)
    return out.cpu().numpy()


def step(grid, q, dt):
    dg = snap.device_grid(grid)
    qd = torch.as_tensor(q).cuda()
    snap.snap_rk3_step(dg, qd, dt, snap.workspace(dg, snap.SNAP_OP_RK3))
    return grid.interior(qd.cpu().numpy())


def close(got, ref, what):
    for v in range(ref.shape[0]):
        scale = np.max(np.abs(ref[v]))
        assert np.max(np.abs(got[v] - ref[v])) <= 1e-12 * scale, (what, v)


@pytest.mark.parametrize("riemann", [0, 1], ids=["lmars", "hllc"])
@pytest.mark.parametrize("nt", [2, 3, 4])
@pytest.mark.parametrize("size", [(17, 9, 9), (33, 20, 6), (16, 16, 5), (7, 5, 8), (20, 24, 7)],
                         ids=lambda s: "x".join(map(str, s)))
def test_both_tiles(size, nt, riemann, monkeypatch):
    print(f"[half tile] {size} nt {nt} riemann {riemann}", flush=True)
    grid, q = case(size, nt, riemann)
    ref, ref1 = oracle.rhs(q, grid).numpy(), grid.interior(oracle.rk3_step(q, grid, 0.05).numpy())
    for half in "01":
        monkeypatch.setenv("SNAP_STAGE_HALF", half)
        close(rhs(grid, q), ref, f"rhs half={half}")
        close(step(grid, q, 0.05), ref1, f"step half={half}")


# narrow last tile, full ones, and with more than a workgroup per compute unit slabs and cubes
@pytest.mark.parametrize("size,half", [((33, 31, 9), True), ((36, 16, 9), True), ((37, 31, 9), False),
                                       ((32, 31, 9), False), ((160, 24, 80), True), ((500, 8, 60), True),
                                       ((100, 100, 100), False)])
def test_rule(size, half, monkeypatch):
    print(f"[half tile] rule {size}", flush=True)
    grid, q = case(size, 2, 0)
    default = rhs(grid, q)
    monkeypatch.setenv("SNAP_STAGE_HALF", "1" if half else "0")
    same = rhs(grid, q)
    monkeypatch.setenv("SNAP_STAGE_HALF", "0" if half else "1")
    other = rhs(grid, q)
    assert np.array_equal(default, same)
    assert not np.array_equal(default, other)   # the two tiles round differently
