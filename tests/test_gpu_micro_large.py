"""Microphysics of a state whose cells fill more than 2^32 threads in blocks of
256: 257 cells by 2^23 levels (62 and 70 GB in single precision), where a launch
with every block along one axis would be refused. Each level holds the same
row, and a cell's result depends on that cell alone, so every level must equal a
single one's bit for bit; and more levels than a launch holds blocks along one of
its other axes, with rows shorter than a block.
"""
import numpy as np
import pytest
import torch

import paper_1901_02955_amd as snap
import workloads as wl

pytestmark = pytest.mark.gpu


def row_case(kind, nx):
    build = wl.jovian_kessler_3d if kind == "kessler" else wl.jovian_satadj_3d
    g, q, params = build(nx=nx, ny=1, nz=12)
    params = type(params)(**{**vars(params), "species": params.species[:1]})
    sp = params.species[0]
    keep = [sp.vapour, sp.cloud] + ([sp.precip] if kind == "kessler" else [])
    names = ["vapour", "cloud"] + (["precip"] if kind == "kessler" else [])
    sp = type(sp)(**{**vars(sp), **{n: i for i, n in enumerate(names)}})
    params = type(params)(**{**vars(params), "species": (sp,)})
    row = g.interior(q)[[0, 1, 2, 3, 4] + [5 + t for t in keep], 5, 0]
    cut = {f: tuple(getattr(g, f)[t] for t in keep) for f in
           ("tracer_kind", "tracer_eps", "tracer_sigma", "tracer_mu")}

    def grid(nz):
        return g.copy(nz=nz, ntracer=len(keep), tracer_wt=(), rhobar_cell=np.ones(nz + 6), pbar_cell=np.ones(nz + 6),
                      rhobar_face=np.ones(nz + 1), pbar_face=np.ones(nz + 1), **cut)

    return grid, torch.as_tensor(np.ascontiguousarray(row)).float().cuda(), params


def run(grid, row, params, kind):
    dg = snap.device_grid(grid, dtype=torch.float32)
    q = torch.empty(dg.shape, dtype=torch.float32, device="cuda")
    inner = q[:, 3:-3, 0, 3:-3]
    inner.copy_(row[:, None, :].expand(inner.shape))
    if kind == "kessler":
        snap.snap_kessler_step(dg, q, 2.0, params)
    else:
        snap.snap_saturation_adjust(dg, q, params)
    return inner


@pytest.mark.parametrize("nx,nz", [(257, 1 << 23), (3, 70000)])
@pytest.mark.parametrize("kind", ["kessler", "saturation"])
def test_every_level(kind, nx, nz):
    print(f"[micro large] {kind} {nx} x {nz}", flush=True)
    torch.cuda.empty_cache()
    grid, row, params = row_case(kind, nx)
    need = 1.2 * row.shape[0] * (nx + 6) * (nz + 6) * 4
    if torch.cuda.mem_get_info()[0] < need:
        pytest.skip(f"needs {need / 1e9:.0f} GB of free device memory")
    ref = run(grid(1), row, params, kind)[:, 0].clone()
    assert torch.isfinite(ref).all() and not torch.equal(ref, row)
    got = run(grid(nz), row, params, kind)
    for v in range(row.shape[0]):
        for k in range(0, nz, 1 << 20):
            assert bool((got[v, k:k + (1 << 20)] == ref[v]).all()), (v, k)
    del got
    torch.cuda.empty_cache()
