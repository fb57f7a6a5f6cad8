"""GPU parity of lstm_int_calibrate: the statistics run of Sec. 4 (float LSTM
of Sec. 2 in double precision on the GPU) against the oracle's float LSTM.

Both sides compute the same real-valued recursion in double; they differ in
the order of the sums (matrix products, layer-norm means), so the comparison
is to a relative 1e-9, far above the rounding of sums of a few thousand
doubles and far below anything that moves a quantization scale."""
import numpy as np
import pytest

import lstm_workloads as wl

pytestmark = pytest.mark.gpu

VARIANTS = [0, wl.LAYER_NORM, wl.PEEPHOLE, wl.PROJECTION, wl.CIFG,
            wl.LAYER_NORM | wl.PEEPHOLE | wl.PROJECTION, wl.CIFG | wl.LAYER_NORM,
            wl.CIFG | wl.LAYER_NORM | wl.PEEPHOLE | wl.PROJECTION]
RTOL = 1e-9


def _close(a, b):
    a, b = np.asarray(a, dtype=np.float64), np.asarray(b, dtype=np.float64)
    assert a.shape == b.shape
    assert np.all(np.abs(a - b) <= RTOL * np.maximum(1.0, np.abs(b))), (a, b)


def _compare(orc, layers, x):
    import torch
    from paper_2101_05453_amd import binding

    y_ref, st_ref = orc.float_forward(layers, x)
    xd = torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()
    st, y = binding.calibrate(layers, xd, want_output=True, apply=False)
    torch.cuda.synchronize()
    _close(y.cpu().numpy(), y_ref)
    assert len(st) == len(st_ref)
    for got, ref in zip(st, st_ref):
        for k in ("x_min", "x_max", "h_min", "h_max", "m_min", "m_max", "c_absmax"):
            _close(got[k], ref[k])
        _close(got["g_absmax"], ref["g_absmax"])
    return st, st_ref


@pytest.mark.parametrize("flags", VARIANTS)
def test_statistics_and_float_output_every_variant(orc, flags):
    # two stacked layers; sizes that are no multiples of the kernels' tiles (16 rows, 64 columns, 32 k)
    layers, x = wl.make_custom([24, 40 if flags & wl.PROJECTION else 72], 72, 40, flags, 5, 7, seed=3)
    _compare(orc, layers, x)


def test_single_row_single_step(orc):
    layers, x = wl.make_custom([8], 16, 16, wl.LAYER_NORM, 1, 1, seed=5)
    _compare(orc, layers, x)


@pytest.mark.parametrize("I,N,H,flags,B,T", [
    (17, 130, 130, wl.LAYER_NORM, 17, 3),  # one row beyond a tile of 16
    (33, 1030, 20, wl.LAYER_NORM | wl.PEEPHOLE | wl.PROJECTION, 40, 2),  # o gate's statistics after the new cell state
    (8, 2050, 16, wl.LAYER_NORM | wl.PROJECTION, 3, 2),  # rows one past a register form of the cell
    (8, 4100, 24, wl.CIFG | wl.LAYER_NORM | wl.PEEPHOLE | wl.PROJECTION, 2, 2),  # rows too wide for registers
    (16, 512, 512, wl.PEEPHOLE, 3, 3),  # few columns, long k: split over 16 waves
    (20, 520, 520, wl.CIFG, 260, 4),  # 128 x 128 blocks with ragged edges on both sides
])
def test_edges_of_the_products_and_of_the_cell(orc, I, N, H, flags, B, T):
    layers, x = wl.make_custom([I], N, H, flags, B, T, seed=N + B)
    _compare(orc, layers, x)


@pytest.mark.parametrize("I,N,H,flags,B,T", [
    (16, 32, 32, wl.LAYER_NORM, 1, 3),                        # one group of 32 columns per gate
    (24, 96, 96, wl.LAYER_NORM | wl.CIFG, 16, 4),
    (24, 160, 48, wl.LAYER_NORM | wl.PROJECTION, 33, 3),      # two rows of tiles per workgroup, the last of one row
    (16, 2080, 40, wl.LAYER_NORM | wl.PROJECTION, 3, 3),      # more than 64 groups per gate: two per lane
    (16, 4096, 33, wl.LAYER_NORM | wl.PROJECTION | wl.CIFG, 2, 2),
    (16, 2048, 64, wl.LAYER_NORM | wl.PROJECTION, 129, 2),    # blocks of 128: the sums from a pass over the row
    (16, 96, 96, wl.LAYER_NORM | wl.PEEPHOLE, 5, 4),          # a gate's sum is not whole before the cell state is
    (16, 64, 64, wl.LAYER_NORM, 256, 3),                      # the last batch with an extreme per thread
    (16, 64, 64, wl.LAYER_NORM, 257, 3),
    (16, 64, 64, 0, 300, 3),
    (16, 516, 17, wl.PROJECTION, 5, 3),                       # a long k over four rows and 16 columns: remainders of all three
    (16, 2048, 640, wl.PROJECTION, 16, 2),
    (16, 3000, 3, wl.PROJECTION, 1, 2),
])
def test_sums_along_with_the_products_and_extremes_over_the_steps(orc, I, N, H, flags, B, T):
    layers, x = wl.make_custom([I], N, H, flags, B, T, seed=N + B)
    _compare(orc, layers, x)


def test_c2_statistics_give_the_same_integer_model(orc):
    """At C2's shape the GPU statistics lead prepare to the very model the
    oracle's statistics lead to: every scale, multiplier and quantized tensor."""
    import torch
    from paper_2101_05453_amd import binding

    layers, x = wl.make_workload("C2")
    rows = np.ascontiguousarray(x[:, :16])
    st, st_ref = _compare(orc, layers, rows)
    orc.apply_stats(layers, st_ref)
    ref = binding.prepare(layers, device=-1).get_quant(0)
    xd = torch.from_numpy(rows.astype(np.float32)).cuda()
    binding.calibrate(layers, xd)  # writes the statistics into the specs
    got = binding.prepare(layers, device=-1).get_quant(0)
    assert got.keys() == ref.keys()
    for k in ref:
        if isinstance(ref[k], np.ndarray):
            assert np.array_equal(got[k], ref[k]), k
        else:
            assert got[k] == ref[k], k


def test_c4_stack_statistics(orc):
    """The 8-layer stack of the headline configuration, on its 16 calibration rows."""
    layers, x = wl.make_workload("C4")
    _compare(orc, layers, np.ascontiguousarray(x[:, :16]))


def test_argument_errors():
    import torch
    from paper_2101_05453_amd import binding

    layers, x = wl.make_custom([8], 16, 16, 0, 2, 2, seed=1)
    xd = torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()
    layers[0].W[1] = None  # a missing gate matrix
    with pytest.raises(binding.LstmIntError):
        binding.calibrate(layers, xd)


def test_more_rows_than_one_launch_takes():
    """2 steps of 4194305 batch rows: one row more than a launch of the cell kernel takes, and T B = 8388610 rows of the
    hoisted product, which are more than 65535 blocks of 128.  One cell, so that the reference is elementwise."""
    import torch
    from paper_2101_05453_amd import binding

    T, B = 2, (1 << 22) + 1
    layers, _ = wl.make_custom([1], 1, 1, 0, 1, 1, seed=4, weight_param=0.5)
    p = layers[0]
    x = torch.randn((T, B, 1), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    st, y = binding.calibrate(layers, x, want_output=True, apply=False)
    h = c = torch.zeros(B, dtype=torch.float64, device="cuda")
    want, cabs = [], 0.0
    for t in range(T):
        i, f, z, o = (float(p.W[g][0, 0]) * x[t, :, 0].double() + float(p.R[g][0, 0]) * h + float(p.b[g][0]) for g in range(4))
        c = torch.sigmoid(i) * torch.tanh(z) + torch.sigmoid(f) * c
        h = torch.sigmoid(o) * torch.tanh(c)
        want.append(h)
        cabs = max(cabs, float(c.abs().max()))
    want = torch.stack(want)
    assert float((y[:, :, 0] - want).abs().max()) <= RTOL
    _close([st[0][k] for k in ("x_min", "x_max", "h_min", "h_max", "c_absmax")],
           [float(x.min()), float(x.max()), float(want.min()), float(want.max()), cabs])
