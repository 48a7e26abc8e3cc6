"""Right-hand-side adjoint with several lines in a wave: lengths at the edges of
four lines (6 and 7 cells) and two (22 and 23) along x, y and z, one cell, and line
counts that leave the last wave and workgroup partly empty. Against the oracle's
autograd, with the tolerances of the longer lines (1e-11 in double and 1e-4 in
single precision of each field's maximum).
"""
import pytest
import torch

import oracle

from tests.test_gpu_adjoint_lanes import adjoint, case, close

pytestmark = pytest.mark.gpu

SIZES = [(6, 7, 22), (7, 22, 6), (22, 6, 7), (23, 5, 3), (5, 23, 7), (17, 2, 23), (1, 5, 22), (22, 1, 5), (33, 6, 1)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("form", [(0, False, 0), (8, False, 0), (6, True, 0), (2, False, 1)],
                         ids=["dry", "tracers8", "mixture6", "hllc2"])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_lines_per_wave(size, form, dtype, monkeypatch):
    print(f"[short lines] {size} {form} {dtype}", flush=True)
    grid, q, rb = case(size, *form, dtype)
    monkeypatch.setenv("SNAP_ADJ_MARCH", "0")
    ref = oracle.rhs_adjoint(q.double().numpy(), grid, rb.double().numpy()).numpy()
    close(adjoint(grid, q, rb), ref, 1e-11 if dtype == torch.float64 else 1e-4)
