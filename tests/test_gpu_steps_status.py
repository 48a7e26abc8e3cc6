"""What snap_rk3_steps_status answers for the state a device-dt call ends with.

The header documents it: the states the steps start from are checked on every
grid, the final one on 3-D grids without tracers only; on other grids the next
call reports it. A step of a smooth state with a Courant number of 1e6 starts
from a good state and ends with one that is not (every kernel runs to its end: none
branches on the values).
"""
import pytest
import torch

import paper_1901_02955_amd as snap
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("ny,nt,riemann", [(1, 0, 0), (1, 0, 1), (1, 3, 0), (9, 2, 0), (9, 0, 0)])
def test_final_state(ny, nt, riemann, dtype):
    print(f"[steps status] ny {ny} tracers {nt} riemann {riemann} {dtype}", flush=True)
    grid, _ = wl.dry_grid(37, ny, 19, 7400.0, 200.0 * ny, 2850.0, bc=(0, 0, 1))
    if ny == 1:
        grid.dy = 1.0
    grid.ntracer, grid.riemann = nt, riemann
    dg = snap.device_grid(grid, dtype=dtype)
    q = torch.as_tensor(wl.random_smooth_state(grid, 17)).to(dtype).cuda()
    work = snap.workspace(dg, snap.SNAP_OP_RK3_CFL)
    snap.snap_rk3_steps_cfl(dg, q, 1e6, 1, work)
    with pytest.raises(snap.SnapError):   # the state itself is bad
        snap.snap_cfl_dt(dg, q, 0.9, snap.workspace(dg, snap.SNAP_OP_CFL))
    if ny > 1 and nt == 0:
        with pytest.raises(snap.SnapError) as err:
            snap.snap_rk3_steps_status(dg, work)
        assert err.value.code == snap.SNAP_E_STATE
    else:
        snap.snap_rk3_steps_status(dg, work)
    snap.snap_rk3_steps_cfl(dg, q, 0.9, 1, work)
    with pytest.raises(snap.SnapError) as err:
        snap.snap_rk3_steps_status(dg, work)
    assert err.value.code == snap.SNAP_E_STATE
