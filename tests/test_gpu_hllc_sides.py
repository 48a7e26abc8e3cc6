"""HLLC with tracers in still air: every face takes the tracers of one side.

At rest the contact speed is zero and the mass flux of a face is what rounding
leaves of it, of either sign, so a rule for the upwind side that looks at the
mass flux need not agree with the flux's own. A face between two tiles is
evaluated in both; if they disagree, the tracer does not leave one as it enters
the other. With uniform pressure, velocity zero and tracers that differ from cell
to cell, the right-hand side of the state moved along the periodic axes must be
the moved right-hand side, bit for bit: a face's flux is the same operations on
the same numbers wherever it lies in a tile (no product of the rest state is
nonzero where two instances could contract a sum differently).
"""
import numpy as np
import pytest
import torch

import paper_1901_02955_amd as snap
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("nt", range(1, 9))
@pytest.mark.parametrize("size", [(48, 40, 12), (48, 1, 40), (112, 96, 40)], ids=lambda s: "x".join(map(str, s)))
def test_moved_state(size, nt, dtype):
    print(f"[hllc sides] {size} nt {nt} {dtype}", flush=True)
    nx, ny, nz = size
    grid, _ = wl.dry_grid(nx, ny, nz, 100.0 * nx, 100.0 * ny, 100.0 * nz, bc=(0, 0, 1))
    if ny == 1:
        grid.dy = 1.0
    grid.ntracer, grid.riemann = nt, 1
    rho, p = (a[3:-3, None, None] * np.ones((1, ny, nx)) for a in (grid.rhobar_cell, grid.pbar_cell))
    rng = np.random.default_rng(nt)
    q = wl.state_from_primitives(grid, rho, 0.0, 0.0, 0.0, p, [rng.random(rho.shape) for _ in range(nt)])
    inner = torch.as_tensor(np.ascontiguousarray(grid.interior(q))).to(dtype).cuda()
    dg = snap.device_grid(grid, dtype=dtype)

    def rhs(x):
        qd = torch.zeros(dg.shape, dtype=dtype, device="cuda")
        grid.interior(qd).copy_(x)
        out = torch.empty(dg.interior_shape, dtype=dtype, device="cuda")
        snap.snap_rhs(dg, qd, out)
        return out

    move = dict(shifts=(3 if ny > 1 else 0, 5), dims=(2, 3))
    a, b = torch.roll(rhs(inner), **move), rhs(torch.roll(inner, **move))
    assert bool(a[5:].any()), "no flux was left by rounding: the test would not see the side"
    assert torch.equal(a, b), [int((a[v] != b[v]).sum()) for v in range(grid.nvar)]
