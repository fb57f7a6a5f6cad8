"""The input matmul of depths 1025 to 2048 (weights in registers, deep_gemm.hip) at its edges: blocks of 32 rows that the
rows do not fill, one block, odd and even numbers of them, parts of the rows without any; both depths it is built for and
depths between; columns that fill no piece of 16, no tile and no workgroup, several gates within a tile, few column blocks and
many; operands that the rescale shifts or clamps first."""
import numpy as np
import pytest

import lstm_workloads as wl
from test_gpu_gru import gru, run_both_paths  # noqa: F401
from test_gpu_sru import compare_all, sru  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("I,N,B,T,weights", [
    (1025, 8, 1, 1, 0.03),       # one row, half a piece per gate
    (1088, 24, 31, 1, 0.03),     # gates begin within a tile
    (1536, 40, 32, 1, 0.03),
    (1537, 40, 33, 1, 0.03),     # two blocks; the deeper form
    (2048, 136, 97, 1, 0.03),    # four blocks, the last with one row
    (2048, 264, 5, 33, 0.03),    # six blocks; nine column blocks
    (1600, 16, 7, 301, 0.03),    # more blocks than parts
    (1088, 1088, 9, 3, 0.03),    # three slots
    (2048, 32, 40, 2, 0.3),      # large scales: the operand is shifted
    (2048, 32, 40, 2, 40.0),     # ... and clamped (the gates' weights only: the state has a largest format)
    (1100, 12, 40, 2, 0.03),     # columns of no whole pieces: the general matmul
    (2112, 16, 40, 2, 0.03),     # deeper than the registers hold: the general matmul
])
def test_sru_input_term(sru, I, N, B, T, weights):  # noqa: F811
    layers, x = wl.make_sru([I], N, B, T, seed=I + N, weight_param=min(weights, 0.3))
    for g in (1, 2):
        layers[0].W[g] *= np.float32(weights / min(weights, 0.3))
    compare_all(sru, layers, x, f"deep{I}x{N}b{B}", calibration_rows=min(B, 8))


@pytest.mark.parametrize("I,N,B,T", [(1025, 20, 3, 11), (1600, 90, 33, 2), (2048, 300, 64, 3)])
def test_gru_input_term(gru, I, N, B, T):  # noqa: F811
    layers, x = wl.make_gru([I], N, B, T, seed=I + N, weight_param=0.03)
    run_both_paths(gru, layers, x, f"deep{I}x{N}b{B}")


def test_x_at_the_end_of_its_buffer(sru):  # noqa: F811
    """Rows are read in place: the last block of 32 rows and the pieces beyond a row's depth reach beyond x."""
    import torch
    from paper_2101_05453_amd import binding

    layers, x = wl.make_sru([1088], 64, 5, 1, seed=2)
    sru.calibrate(layers, x, threads=8)
    m = binding.sru_prepare(layers, device=0)
    x8 = np.random.default_rng(3).integers(-128, 128, size=x.shape).astype(np.int8)
    for offset in (0, 8):  # 8: not on a 16-byte boundary, copied first
        buf = torch.zeros(offset + x8.size, dtype=torch.int8, device="cuda")
        xd = buf[offset:].view(*x8.shape)
        xd.copy_(torch.from_numpy(x8))
        m.set_option("register_gemm", 0)
        want = m.forward(xd)
        m.set_option("register_gemm", 1)
        assert torch.equal(m.forward(xd), want)
