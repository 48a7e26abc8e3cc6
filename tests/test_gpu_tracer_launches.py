"""Tracers in every kernel instance that the size of a launch selects, under both
Riemann solvers: 3-D right-hand sides of fewer workgroups than compute units, of up to
twice as many, and of more, for each count of tracers in both precisions, against the
oracle (1e-12 and 1e-4 of each field's maximum, as for every right-hand side).
"""
import pytest
import torch

from tests.test_gpu_tracers import check

pytestmark = pytest.mark.gpu

# 16-cell tiles of 8 x 8 columns: levels for at most 256, 512 and more workgroups
SIZES = {"few": (17, 15, 9), "some": (113, 20, 80), "many": (113, 97, 40)}


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("riemann", [0, 1], ids=["lmars", "hllc"])
@pytest.mark.parametrize("nt", range(1, 9))
@pytest.mark.parametrize("launch", SIZES)
def test_instances(launch, nt, riemann, dtype):
    if launch != "few" and nt > 5:
        pytest.skip("these counts have one instance")
    check(*SIZES[launch], nt, dtype, riemann, (nt % 2, 1, 1))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("riemann", [0, 1], ids=["lmars", "hllc"])
@pytest.mark.parametrize("nt", range(1, 9))
def test_flat(nt, riemann, dtype):
    check(31, 1, 18, nt, dtype, riemann, (nt % 2, 0, 1))
