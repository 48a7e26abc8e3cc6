"""Conservation sums of states that take every block several passes, with
remainders: rows of one cell up to rows longer than a block's threads, in both
precisions and both storage forms, against the sums in extended precision.

A pass covers 512 blocks of 1024 threads, and the sizes below need two or three.
Each value passes through at most 3 additions of its thread, 6 of the wave, 16 of
the block, and 2 + 6 + 4 over the blocks, and the added references of the
perturbation form through 3 more roundings: 40 of 2^-53 each, 4.5e-15 of the sum
of magnitudes.
"""
import numpy as np
import pytest
import torch

import paper_1901_02955_amd as snap
import workloads as wl

pytestmark = pytest.mark.gpu

SIZES = [(1, 900, 700), (2, 1, 300000), (3, 500, 300), (33, 97, 100), (64, 100, 83), (1025, 20, 15), (300, 41, 37)]


@pytest.mark.parametrize("storage", ["total", "perturbation"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("nt", [0, 8])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_many_passes(size, nt, dtype, storage):
    nx, ny, nz = size
    print(f"[sums passes] {size} tracers {nt} {dtype} {storage}", flush=True)
    grid, _ = wl.dry_grid(nx, ny, nz, 200.0 * nx, 200.0 * ny, min(150.0, 12e3 / nz) * nz, bc=(0, 0, 1))
    grid.ntracer = nt
    rng = np.random.default_rng(nx + nt)
    q = torch.as_tensor(rng.standard_normal(grid.shape, dtype=np.float32)).to(dtype)
    form = snap.SNAP_STORE_TOTAL if storage == "total" else snap.SNAP_STORE_PERTURBATION
    dg = snap.device_grid(grid, dtype=dtype, storage=form)
    got = snap.snap_conservation_sums(dg, q.cuda(), snap.workspace(dg, snap.SNAP_OP_SUMS))
    vals = grid.interior(q.numpy()).astype(np.longdouble)
    if storage == "perturbation":
        vals[0] += grid.rhobar_cell[3:-3, None, None]
        vals[4] += grid.pbar_cell[3:-3, None, None].astype(np.longdouble) / (grid.gamma - 1.0)
    vals = vals.reshape(grid.nvar, -1)
    assert np.all(np.abs(got - vals.sum(axis=1)) <= 4.5e-15 * np.abs(vals).sum(axis=1))
