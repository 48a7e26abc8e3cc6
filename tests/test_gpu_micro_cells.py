"""The microphysics kernels take each cell by itself: the same cells on another
grid give the same bits.

A level's cells are dealt to blocks of 256 in one run over its rows, so levels
of fewer cells than a block, of exactly one block, and of several with a
remainder are compared, 2-D rows included, for the Kessler step, the saturation
adjustment and their adjoints, with one species and with two (the iteration
keeps the species it has in registers). The small grids' results are held
against the oracle elsewhere; here the tolerance is zero.
"""
import numpy as np
import pytest
import torch

import paper_1901_02955_amd as snap
import workloads as wl

pytestmark = pytest.mark.gpu

# cells in all: 23 * 13 * 12; planes of 299, 156, 256-cell remainders and rows
BASE = (13, 12, 23)
SHAPES = [(23, 13, 12), (299, 1, 12), (3588, 1, 1), (1, 276, 13), (26, 138, 1)]


def rearranged(g, q, shape):
    nx, ny, nz = shape
    h = g.copy(nx=nx, ny=ny, nz=nz, rhobar_cell=np.ones(nz + 6), pbar_cell=np.ones(nz + 6),
               rhobar_face=np.ones(nz + 1), pbar_face=np.ones(nz + 1))
    p = np.ones(h.shape)
    h.interior(p)[...] = g.interior(q).reshape(h.interior_shape)
    return h, p


def run(g, q, kind, params, species, dtype):
    p = type(params)(**{**vars(params), "species": params.species[:species]})
    dg = snap.device_grid(g, dtype=dtype)
    qd = torch.as_tensor(q).to(dtype).cuda()
    qb = torch.linspace(-1.0, 1.0, int(np.prod(g.interior_shape)), dtype=dtype,
                        device="cuda").reshape(g.interior_shape)
    if kind == "kessler":
        snap.snap_kessler_step_adjoint(dg, qd, 2.0, p, qb)
        snap.snap_kessler_step(dg, qd, 2.0, p)
    else:
        snap.snap_saturation_adjust_adjoint(dg, qd, p, qb)
        snap.snap_saturation_adjust(dg, qd, p)
    out = g.interior(qd.cpu().numpy()).reshape(g.nvar, -1)
    ghosts = qd.cpu().numpy().copy()
    g.interior(ghosts)[...] = 1.0
    return out, qb.cpu().numpy().reshape(g.nvar, -1), ghosts


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("species", [1, 2])
@pytest.mark.parametrize("kind", ["kessler", "saturation"])
def test_cells_alone(kind, species, dtype):
    nx, ny, nz = BASE
    build = wl.jovian_kessler_3d if kind == "kessler" else wl.jovian_satadj_3d
    g, q, params = build(nx=nx, ny=ny, nz=nz)
    ref = run(g, q, kind, params, species, dtype)
    assert np.isfinite(ref[0]).all() and np.isfinite(ref[1]).all()
    for shape in SHAPES:
        print(f"[micro cells] {kind} {species} {dtype} {shape}", flush=True)
        h, p = rearranged(g, q, shape)
        got = run(h, p, kind, params, species, dtype)
        assert np.array_equal(got[0], ref[0]), shape
        assert np.array_equal(got[1], ref[1]), shape
        assert (got[2] == 1.0).all(), shape
