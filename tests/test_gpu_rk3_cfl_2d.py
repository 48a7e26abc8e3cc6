"""Device-dt steps in 2-D, whose last stage reduces the next step's signal speed:
every dt and state of four steps in one call equals, bit for bit, snap_cfl_dt and
snap_rk3_step in turn. Moving states with dx different from dz on ragged tiles,
walls and periodic axes, tracers, HLLC, the perturbation form, both precisions.
"""
import numpy as np
import pytest
import torch

import paper_1901_02955_amd as snap
import workloads as wl

pytestmark = pytest.mark.gpu

CFL = 0.9


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("storage", ["total", "perturbation"])
@pytest.mark.parametrize("riemann", [0, 1], ids=["lmars", "hllc"])
@pytest.mark.parametrize("nt", [0, 3])
@pytest.mark.parametrize("size,bc", [((37, 19), (1, 0, 1)), ((64, 48), (0, 0, 1)), ((17, 33), (0, 0, 0)), ((2, 5), (1, 0, 1))])
def test_steps(size, bc, nt, riemann, storage, dtype):
    print(f"[rk3-cfl 2d] {size} bc {bc} nt {nt} riemann {riemann} {storage} {dtype}", flush=True)
    nx, nz = size
    grid, _ = wl.dry_grid(nx, 1, nz, 310.0 * nx, 1.0, 140.0 * nz, bc=bc)
    grid.dy, grid.ntracer, grid.riemann = 1.0, nt, riemann
    q = wl.random_smooth_state(grid, 70 + nx)
    form = snap.SNAP_STORE_TOTAL
    if storage == "perturbation":
        q, form = wl.to_perturbation(grid, q), snap.SNAP_STORE_PERTURBATION
    dg = snap.device_grid(grid, dtype=dtype, storage=form)
    host = torch.as_tensor(np.asarray(q)).to(dtype).cuda()
    dev = host.clone()
    work, cw = snap.workspace(dg, snap.SNAP_OP_RK3), snap.workspace(dg, snap.SNAP_OP_CFL)
    dts = []
    for _ in range(4):
        dts.append(snap.snap_cfl_dt(dg, host, CFL, cw))
        snap.snap_rk3_step(dg, host, dts[-1], work)
    out = torch.full((4,), -1.0, dtype=torch.float64, device="cuda")
    wcfl = snap.workspace(dg, snap.SNAP_OP_RK3_CFL)
    snap.snap_rk3_steps_cfl(dg, dev, CFL, 4, wcfl, out)
    snap.snap_rk3_steps_status(dg, wcfl)
    assert len(set(dts)) == 4
    assert out.cpu().tolist() == dts
    assert torch.equal(grid.interior(dev), grid.interior(host))
