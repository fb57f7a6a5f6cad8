"""The persistent kernels of the integer GRU at the edges of their tiles and of their dispatch: carried state over two
calls, on the one-launch form and on the launch-per-step form, against the CPU oracle."""
import pytest

import lstm_workloads as wl
from test_gpu_gru import gru, run_both_paths  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inputs,N,B,T", [
    # groups of four rows
    ([20], 64, 5, 6),             # one workgroup per group: no exchange
    ([20], 65, 3, 4),             # a second workgroup with one cell
    ([20], 130, 7, 300),          # the tags wrap at 256 steps
    ([20], 513, 6, 4),
    ([20], 1100, 4, 3),
    ([20, 1203], 1203, 5, 3),     # row-major input terms, a last piece of them beyond the columns
    ([20, 2048], 2048, 32, 3),    # every compute unit
    # groups of 16 rows
    ([20], 60, 1030, 3),
    ([20], 300, 195, 4),
    ([20], 1024, 65, 3),
    ([20, 1203], 1203, 37, 3),
    ([20, 2048], 2048, 113, 3),
    # groups of 32 rows
    ([20], 257, 780, 3),
    ([20, 1203], 1203, 140, 3),
    ([20], 2047, 256, 3),
    ([20, 2048], 2048, 290, 2),   # a second launch
])
def test_edges_of_the_persistent_kernels(gru, inputs, N, B, T):  # noqa: F811
    layers, x = wl.make_gru(inputs, N, B, T, seed=N + B, weight_param=0.9 / N ** 0.5, input_param=1.5)
    rows = None if B <= 16 else sorted({0, 1, 15, 16, 31, min(32, B - 1), B // 2, B - 2, B - 1})
    run_both_paths(gru, layers, x, f"gru{inputs}x{N}b{B}", rows=rows, splits=[(0, 1), (1, T)])


@pytest.mark.parametrize("inputs,N,B,T", [
    ([20], 64, 1030, 7),          # 16 rows, one workgroup per group; the second half of the depth is empty
    ([20], 64, 4100, 7),          # 32 rows of the same, the last group of four rows
    ([20], 130, 1300, 8),         # the input terms of four turns and more through three places
    ([20], 520, 500, 7),          # nine k steps: eight and one
    ([20, 1203], 1203, 150, 7),   # row-major input terms
])
def test_halves_of_the_depth_and_turns_of_the_tiles(gru, inputs, N, B, T):  # noqa: F811
    layers, x = wl.make_gru(inputs, N, B, T, seed=N + B, weight_param=0.9 / N ** 0.5, input_param=1.5)
    rows = sorted({0, 15, 16, 31, 32, B // 2, B - 3, B - 1})
    run_both_paths(gru, layers, x, f"halves{inputs}x{N}b{B}", rows=rows)


@pytest.mark.parametrize("B", [40, 1100])
def test_waits_give_up_and_the_model_recovers(gru, B):  # noqa: F811
    """Both exchanges: with the test hook a wait ends at its limit and the status word says so."""
    import torch
    from paper_2101_05453_amd import binding

    layers, x = wl.make_gru([32], 96, B, 5, seed=9, weight_param=0.2)
    m = binding.gru_prepare(layers, device=0)
    xd = torch.randint(-128, 128, (5, B, 32), dtype=torch.int8, device="cuda")
    want = m.forward(xd)
    m.set_option("spin_limit", 64)
    m.set_option("barrier_never_completes", 1)
    m.forward(xd)
    assert m.device_status() == 1
    m.set_option("barrier_never_completes", 0)
    m.set_option("spin_limit", 1 << 21)
    m.set_option("reset_status", 1)
    assert torch.equal(m.forward(xd), want) and m.device_status() == 0


@pytest.mark.parametrize("T", [1, 2, 4, 6, 13])
@pytest.mark.parametrize("N,B", [(130, 520), (600, 110), (130, 2060), (600, 400)])  # 16 rows, 32 rows
def test_slots_of_the_exchange_in_turn(gru, N, B, T):  # noqa: F811
    layers, x = wl.make_gru([20, N], N, B, T, seed=N + T, weight_param=0.9 / N ** 0.5, input_param=1.5)
    rows = sorted({0, 15, 16, 31, 32, B // 2, B - 3, B - 1})
    run_both_paths(gru, layers, x, f"slots{N}b{B}t{T}", rows=rows)


@pytest.mark.parametrize("B", [300, 1030])  # groups of 16 and of 32 rows
@pytest.mark.parametrize("T", [1, 3, 9])
def test_states_that_look_like_marks(gru, B, T):  # noqa: F811
    """Cells at both ends of the range by turns, every eighth of them to either side of -127."""
    import numpy as np
    import torch
    from test_gpu_gru import both, equal, quantize_x

    N = 200
    layers, x = wl.make_gru([20], N, B, T, seed=3, weight_param=0.01)
    n = np.arange(N)
    layers[0].bx[1][:] = -6.0  # the state is the candidate
    layers[0].bx[2][:] = np.where(n % 8 == 0, -2.2 - 2.2 * n / N, np.where(n % 2, 6.0, -6.0))
    m, old = both(gru, layers)
    xq = quantize_x(x, old.get_quant(0))
    rows = sorted({0, 15, 16, 31, 32, B - 1})
    y = m.forward(torch.from_numpy(xq).cuda())
    assert m.device_status() == 0
    want, trace = old.forward(np.ascontiguousarray(xq[:, rows]), trace_layer=0)
    words = np.ascontiguousarray(trace["h8"]).view(np.uint32)[:, :, ::2]
    assert (words == 0x7F807F80).any() and (words == 0x7F807F81).any()
    equal("y", y.cpu().numpy()[:, rows], want)
