"""The SRU scan with the table of all sigma values (large batches, eight steps and more): the smallest call that takes it,
the largest ones that do not, and a ragged one."""
import pytest

import lstm_workloads as wl
from test_gpu_sru import compare_all, sru  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inputs,N,B,T", [
    ([64], 1024, 320, 8),  # 320 workgroups of the other form
    ([64], 1024, 320, 7),  # too few steps
    ([64], 1024, 288, 8),  # too few workgroups
    ([64, 1028], 1028, 330, 9),  # tile order, then row-major
    ([64], 1024, 256, 8),
    ([64], 1024, 256, 7),
    ([64, 1028], 1028, 257, 9),
])
def test_scan_with_the_full_table(sru, inputs, N, B, T):  # noqa: F811
    layers, x = wl.make_sru(inputs, N, B, T, seed=N + T, weight_param=0.04, input_param=2.0)
    compare_all(sru, layers, x, f"sru{N}x{B}x{T}", rows=[0, 31, 32, 255, B - 1], calibration_rows=16)
