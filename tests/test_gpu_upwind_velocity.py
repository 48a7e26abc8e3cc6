"""Right-hand side of rough double-precision 3-D flows, whose tangential
velocities are reconstructed on the upwind side of each face only, against the
oracle, which reconstructs both sides of every variable.

Every velocity component changes from cell to cell by more than its mean, so
that the upwind side alternates along each axis and the two sides' tangential
velocities differ by their own size; one cell beyond and short of the 16-cell
tiles, walls and periodic axes, no tracers and the counts that share the kernel,
linear and nonlinear weights. A resting normal velocity (u* from the pressure
alone) is the second state. Tolerance as for every double-precision right-hand
side: 1e-12 of each field's maximum.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_02955_amd as snap
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", [snap.SNAP_STORE_TOTAL, snap.SNAP_STORE_PERTURBATION],
                         ids=["total", "perturbation"])
@pytest.mark.parametrize("rest", [None, 1, 2, 3], ids=["rough", "u0", "v0", "w0"])
@pytest.mark.parametrize("nx,ny,nz,nt,linear", [(17, 15, 9, 0, False), (33, 16, 4, 1, False),
                                                (16, 31, 5, 5, False), (15, 18, 8, 0, True)])
def test_rough_flow(nx, ny, nz, nt, linear, rest, storage):
    if storage == snap.SNAP_STORE_PERTURBATION and nt:
        nt = 1
    print(f"[upwind velocity] {nx}x{ny}x{nz} nt {nt} rest {rest} storage {storage}", flush=True)
    grid, _ = wl.dry_grid(nx, ny, nz, 200.0 * nx, 200.0 * ny, 150.0 * nz, bc=(nx % 2, ny % 2, 1))
    grid.ntracer, grid.weno_linear = nt, linear
    q = wl.random_smooth_state(grid, 300 + nx)
    rng = np.random.default_rng(nx)
    qi = grid.interior(q)
    old = 0.5 * (qi[1] ** 2 + qi[2] ** 2 + qi[3] ** 2) / qi[0]
    for v in (1, 2, 3):
        qi[v] = 0.0 if v == rest else qi[0] * rng.uniform(-30.0, 30.0, size=qi[0].shape)
    qi[4] += 0.5 * (qi[1] ** 2 + qi[2] ** 2 + qi[3] ** 2) / qi[0] - old
    dg = snap.device_grid(grid, dtype=torch.float64, storage=storage)
    stored = q.copy()
    if storage == snap.SNAP_STORE_PERTURBATION:
        si = grid.interior(stored)
        si[0] -= grid.rhobar_cell[3:-3, None, None]
        si[4] -= grid.pbar_cell[3:-3, None, None] / (grid.gamma - 1.0)
    rhs = torch.empty(dg.interior_shape, dtype=torch.float64, device="cuda")
    snap.snap_rhs(dg, torch.as_tensor(stored).cuda(), rhs)
    ref = oracle.rhs(q, grid).numpy()
    got = rhs.cpu().numpy()
    for v in range(grid.nvar):
        scale = np.max(np.abs(ref[v]))
        assert np.max(np.abs(got[v] - ref[v])) <= 1e-12 * scale, (v, np.max(np.abs(got[v] - ref[v])) / scale)
