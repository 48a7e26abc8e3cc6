"""Right-hand-side adjoint with the cells of a line in the lanes of a wave: line
lengths around the segments a wave holds (54 cells, 57 at an end of the line,
one, two and three segments) along x, y and z, walls and periodic, with the
fewest and the most variables, the mixture and HLLC; and the single-precision
march on the same grids. Against the oracle's autograd.

Tolerances as for every right-hand-side adjoint: 1e-11 (double) and 1e-4
(single precision) of each field's maximum; the march within 1e-5 of the lane
kernel (the same contributions in another order).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_02955_amd as snap
import workloads as wl

pytestmark = pytest.mark.gpu

SIZES = [(53, 3, 4), (54, 2, 7), (55, 4, 3), (109, 1, 5), (3, 54, 8), (5, 55, 3), (2, 109, 4), (4, 3, 54),
         (9, 7, 55), (6, 1, 108), (3, 4, 163)]


def case(size, nt, mixture, riemann, dtype):
    nx, ny, nz = size
    bc = (nx % 2, ny % 2, 1)
    # levels thin enough that the column stays below the isentropic base's top
    grid, base = wl.dry_grid(nx, ny, nz, 200.0 * nx, 200.0 * ny, min(150.0, 12e3 / nz) * nz, bc=bc)
    if ny == 1:
        grid.dy = 1.0
    grid.ntracer, grid.riemann = nt, riemann
    if mixture:
        table = wl.condensable_species(base.cp - base.rd, wl.RGAS / base.rd)
        grid = wl.with_mixture(grid, [table[i % 4] for i in range(nt)])
    q = torch.as_tensor(wl.random_smooth_state(grid, 7 + nx + nt)).to(dtype)
    rb = torch.as_tensor(wl.seeded_normal(grid.interior_shape, 11)).to(dtype)
    return grid, q, rb


def adjoint(grid, q, rb):
    dg = snap.device_grid(grid, dtype=q.dtype)
    out = torch.empty(dg.interior_shape, dtype=q.dtype, device="cuda")
    snap.snap_rhs_adjoint(dg, q.cuda(), rb.cuda(), out, snap.workspace(dg, snap.SNAP_OP_RHS_ADJ))
    return out.double().cpu().numpy()


def close(got, ref, tol):
    for v in range(ref.shape[0]):
        scale = np.max(np.abs(ref[v]))
        assert np.max(np.abs(got[v] - ref[v])) <= tol * scale, (v, np.max(np.abs(got[v] - ref[v])) / scale)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_line_lengths(size, dtype, monkeypatch):
    n = SIZES.index(size)
    nt, mixture, riemann = [(0, False, 0), (8, False, 0), (6, True, 0), (2, False, 1)][n % 4]
    print(f"[lanes] {size} {dtype} nt {nt} mixture {mixture} riemann {riemann}", flush=True)
    grid, q, rb = case(size, nt, mixture, riemann, dtype)
    monkeypatch.setenv("SNAP_ADJ_MARCH", "0")
    got = adjoint(grid, q, rb)
    ref = oracle.rhs_adjoint(q.double().numpy(), grid, rb.double().numpy()).numpy()
    close(got, ref, 1e-11 if dtype == torch.float64 else 1e-4)


@pytest.mark.parametrize("size", SIZES[3:], ids=lambda s: "x".join(map(str, s)))
def test_march(size, monkeypatch):
    print(f"[lanes] march {size}", flush=True)
    grid, q, rb = case(size, SIZES.index(size) % 3, False, 0, torch.float32)
    monkeypatch.setenv("SNAP_ADJ_MARCH", "0")
    lanes = adjoint(grid, q, rb)
    monkeypatch.setenv("SNAP_ADJ_MARCH", "1")
    close(adjoint(grid, q, rb), lanes, 1e-5)
