"""Conservation sums on rows around the kernel's stretch lengths (64 .. 1024
cells, longer rows in several stretches), with the fewest and the most
variables, against the sums of the data in extended precision.

A thread adds at most a few hundred values and the trees a dozen more, each
addition within 2^-53 of its result: 1e-13 of the sum of magnitudes.
"""
import numpy as np
import pytest
import torch

import paper_1901_02955_amd as snap
import workloads as wl

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 8), (63, 5, 7), (64, 3, 4), (65, 1, 9), (1024, 2, 3), (1025, 1, 6), (2500, 3, 5)]


@pytest.mark.parametrize("nt", [0, 8])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_sums(size, nt):
    nx, ny, nz = size
    print(f"[sums] {size} tracers {nt}", flush=True)
    grid, _ = wl.dry_grid(nx, ny, nz, 200.0 * nx, 200.0 * ny, 150.0 * nz, bc=(0, 0, 1))
    grid.ntracer = nt
    q = np.random.default_rng(nx + nt).standard_normal(grid.shape)
    dg = snap.device_grid(grid)
    got = snap.snap_conservation_sums(dg, torch.as_tensor(q).cuda(),
                                      snap.workspace(dg, snap.SNAP_OP_SUMS))
    vals = grid.interior(q).reshape(grid.nvar, -1).astype(np.longdouble)
    bound = 1e-13 * np.abs(vals).sum(axis=1)
    assert np.all(np.abs(got - vals.sum(axis=1)) <= bound), (got, vals.sum(axis=1))
