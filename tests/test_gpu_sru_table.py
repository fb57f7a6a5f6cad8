"""The SRU scan with the table of all sigma values (large batches): calls on both sides of its rule for row-major and for
tile-ordered terms, and ragged ones."""
import pytest

import lstm_workloads as wl
from test_gpu_sru import compare_all, sru  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inputs,N,B,T", [
    ([64], 1024, 320, 8),
    ([64], 1024, 320, 7),
    ([64], 1024, 288, 8),
    ([64, 1028], 1028, 330, 9),  # tile order, then row-major with the table
    ([64], 1024, 256, 8),
    ([64], 1024, 256, 7),
    ([64, 1028], 1028, 257, 9),
    ([1040, 1040], 1040, 252, 3),  # row-major: 256 workgroups of the other form
    ([1040, 1040], 1040, 253, 2),  # and 257
    ([1100], 1040, 253, 1),  # the same with a highway matrix
    ([64, 1024], 1024, 768, 5),  # tile order: the last round with a compute unit per small workgroup
    ([64, 1024], 1024, 790, 6),  # and with more of them than that
])
def test_scan_with_the_full_table(sru, inputs, N, B, T):  # noqa: F811
    layers, x = wl.make_sru(inputs, N, B, T, seed=N + T, weight_param=0.04, input_param=2.0)
    compare_all(sru, layers, x, f"sru{N}x{B}x{T}", rows=sorted({0, 31, 32, min(255, B - 1), B - 1}), calibration_rows=16)
