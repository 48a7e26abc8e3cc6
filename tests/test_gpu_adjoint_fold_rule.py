"""The fold in the z direction against the separate fold pass, on grids on either
side of the rule that picks one (1024 blocks of 256 cells of a row) and on small
ones where it is asked for: walls and periodic axes, 2-D and 3-D, up to eight tracers,
HLLC. The same contributions in another order: within 1e-13 (double) and 1e-5
(single precision) of each field's maximum; and the default is one of the two, bit for
bit.
"""
import numpy as np
import pytest
import torch

from tests.test_gpu_adjoint_lanes import adjoint, case, close

pytestmark = pytest.mark.gpu

# (nx, ny, nz), whether the rule folds: 32 x 32 rows, 31 x 33, two blocks per row
GRIDS = [((20, 38, 38), True), ((20, 37, 39), False), ((257, 22, 38), True), ((40, 1, 1030), True),
         ((40, 1, 1029), False), ((33, 5, 40), False), ((16, 16, 16), False)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("form", [(0, False, 0), (8, False, 0), (2, False, 1)], ids=["dry", "tracers8", "hllc2"])
@pytest.mark.parametrize("size,folds", GRIDS, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else None)
def test_fold(size, folds, form, dtype, monkeypatch):
    print(f"[fold rule] {size} {form} {dtype}", flush=True)
    grid, q, rb = case(size, *form, dtype)
    monkeypatch.setenv("SNAP_ADJ_MARCH", "0")
    default = adjoint(grid, q, rb)
    monkeypatch.setenv("SNAP_ADJ_MARCH_FOLD", "0")
    separate = adjoint(grid, q, rb)
    monkeypatch.setenv("SNAP_ADJ_MARCH_FOLD", "1")
    folded = adjoint(grid, q, rb)
    close(folded, separate, 1e-13 if dtype == torch.float64 else 1e-5)
    assert np.array_equal(default, folded if folds else separate)
