"""Right-hand side with passive tracers, one upwind value per face, against the
oracle: every tracer count (each has kernel instances of its own) on a grid of
ragged tiles, and the counts whose instance depends on the size of the launch on
one with more workgroups than compute units; one cell beyond and short of the
16-cell tiles, walls and periodic axes, LMARS and HLLC, 2-D and 3-D.

Tolerances as for every right-hand side: 1e-12 (double) and 1e-4 (single
precision) of each field's maximum.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_02955_amd as snap
import workloads as wl

pytestmark = pytest.mark.gpu


def check(nx, ny, nz, nt, dtype, riemann, bc, linear=False):
    print(f"[tracers] {nx}x{ny}x{nz} nt {nt} {dtype} riemann {riemann}", flush=True)
    grid, _ = wl.dry_grid(nx, ny, nz, 200.0 * nx, 200.0 * ny, 150.0 * nz, bc=bc)
    if ny == 1:
        grid.dy = 1.0
    grid.ntracer, grid.riemann, grid.weno_linear = nt, riemann, linear
    q = wl.random_smooth_state(grid, 100 + nt)
    dg = snap.device_grid(grid, dtype=dtype)
    qd = torch.as_tensor(q).to(dtype).cuda()
    rhs = torch.empty(dg.interior_shape, dtype=dtype, device="cuda")
    snap.snap_rhs(dg, qd, rhs)
    ref = oracle.rhs(torch.as_tensor(q).to(dtype).double().numpy(), grid).numpy()
    got = rhs.double().cpu().numpy()
    tol = 1e-12 if dtype == torch.float64 else 1e-4
    for v in range(grid.nvar):
        scale = np.max(np.abs(ref[v]))
        assert np.max(np.abs(got[v] - ref[v])) <= tol * scale, (v, np.max(np.abs(got[v] - ref[v])) / scale)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("nt", range(1, 9))
def test_every_count(nt, dtype):
    check(17, 15, 9, nt, dtype, nt % 2, (nt % 2, 0, 1))
    check(31, 1, 18, nt, dtype, (nt + 1) % 2, (nt % 2, 0, 1), linear=nt == 3)


@pytest.mark.parametrize("dtype,nt", [(torch.float64, 3), (torch.float64, 4), (torch.float32, 2),
                                      (torch.float32, 3), (torch.float32, 5)],
                         ids=["f64-3", "f64-4", "f32-2", "f32-3", "f32-5"])
def test_full_launch(dtype, nt):
    check(113, 97, 40, nt, dtype, 0, (0, 1, 1))
