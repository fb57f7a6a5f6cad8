"""Layers of up to 256 cells with a workgroup per batch row: step counts around the ring of W x terms, every combination of options
in each of the three forms, widths that leave lanes and waves without cells, the last batch of that kernel and the first of the
four-row one (whose variants run here too), and both directions of a bidirectional layer in one launch on either side."""
import numpy as np
import pytest

import lstm_workloads as wl
from paper_2101_05453_amd import binding
from parity_util import assert_equal, calibrate_on_gpu, prepare_both, run_and_compare

pytestmark = pytest.mark.gpu
LN, PH, PROJ, CIFG = wl.LAYER_NORM, wl.PEEPHOLE, wl.PROJECTION, wl.CIFG


@pytest.mark.parametrize("N,H", [(5, 5), (64, 64), (50, 33), (65, 65), (128, 100), (100, 128), (129, 129), (200, 256), (256, 80)])
@pytest.mark.parametrize("T", [1, 8, 9, 17, 36])
def test_steps_around_the_ring(orc, N, H, T):
    flags = ((0, LN, PH | LN, CIFG | LN)[T % 4]) | (PROJ if N != H else 0)
    layers, x = wl.make_custom([24, H], N, H, flags, 3, T, seed=N + T, weight_param=0.9 / N ** 0.5)
    run_and_compare(orc, layers, x, f"row{N}h{H}t{T}", trace=False, options={"stack": 0})


@pytest.mark.parametrize("flags", range(16))
@pytest.mark.parametrize("N", [40, 120, 250])
@pytest.mark.parametrize("B", [2, 259])
def test_every_variant(orc, N, B, flags):
    H = N - 9 if flags & PROJ else N
    layers, x = wl.make_custom([32], N, H, flags, B, 5, seed=N + flags, weight_param=0.9 / N ** 0.5)
    run_and_compare(orc, layers, x, f"row{N}b{B}f{flags}", trace=False, rows=sorted({0, 1, B // 2, B - 2, B - 1}))


@pytest.mark.parametrize("N,flags", [(64, LN), (100, PH | LN), (256, 0), (203, PH | LN | PROJ)])
def test_last_batch_of_a_row_per_workgroup(orc, N, flags):
    import torch

    layers, x = wl.make_custom([40], N, N - 3 if flags & PROJ else N, flags, 257, 11, seed=N, weight_param=0.9 / N ** 0.5)
    lib_model, orc_model, xq = prepare_both(orc, layers, x)
    rows = [0, 1, 4, 127, 128, 251, 254, 255]
    want = np.asarray(orc.forward(orc_model, np.ascontiguousarray(xq[:, rows])))
    for B in (255, 256, 257):
        y = lib_model.forward(torch.from_numpy(np.ascontiguousarray(xq[:, :B])).cuda()).cpu().numpy()
        at = [i for i, r in enumerate(rows) if r < B]
        assert_equal(f"y B={B}", y[:, [rows[i] for i in at]], want[:, at])
    assert lib_model.device_status() == 0


@pytest.mark.parametrize("B", [1, 128, 129])
def test_two_directions(orc, B):
    import torch

    layers, x = wl.make_custom([40], 96, 96, LN, B, 19, seed=5, weight_param=0.09)
    back, _ = wl.make_custom([40], 96, 96, LN, B, 19, seed=6, weight_param=0.09)
    fwd, ofwd, xq = prepare_both(orc, layers, x)
    bwd, obwd, _ = prepare_both(orc, back, x)
    q = bwd.get_quant(0)
    if (q["s_x"], q["zp_x"]) != (fwd.get_quant(0)["s_x"], fwd.get_quant(0)["zp_x"]):
        pytest.skip("the two directions read one quantized input")
    bwd.set_option("reverse", 1)
    y = binding.forward_bidirectional(fwd, bwd, torch.from_numpy(xq).cuda()).cpu().numpy()
    rows = sorted({0, B // 2, B - 1})
    xs = np.ascontiguousarray(xq[:, rows])
    assert_equal("forward", y[:, rows, :96], np.asarray(orc.forward(ofwd, xs)))
    assert_equal("backward", y[:, rows, 96:], np.asarray(orc.forward(obwd, np.ascontiguousarray(xs[::-1])))[::-1])


@pytest.mark.parametrize("N,T", [(48, 15), (48, 16), (64, 17), (64, 33), (30, 64), (30, 65), (128, 16), (100, 31), (128, 48), (250, 16), (250, 17)])
@pytest.mark.parametrize("I", [16, 48, 75, 208])
def test_input_product_in_the_launch(orc, N, T, I):
    """W x of up to 64 steps (up to 128 cells, few weights) or 16 steps in the recurrent launch: chunks of 16 steps, rows of x in
    place and through the padded copy, depths that end within a 64-byte step; else the input GEMM."""
    flags = (LN, 0, PH | LN | PROJ, CIFG)[(N + T + I) % 4]
    layers, x = wl.make_custom([I, N], N, N, flags, 5, T, seed=N + T + I, weight_param=0.9 / N ** 0.5)
    run_and_compare(orc, layers, x, f"rowin{N}t{T}i{I}", trace=False, options={"stack": 0})


def test_input_product_counts(orc):
    """On which side of the rule a call is, by the launches of the input GEMM."""
    import torch

    layers, x = wl.make_custom([64], 64, 64, 0, 2, 80, seed=3, weight_param=0.1)
    model, _, xq = prepare_both(orc, layers, x)
    for T, launches in ((1, 0), (16, 0), (32, 0), (80, 1)):
        model.profile_begin()
        model.forward(torch.from_numpy(np.ascontiguousarray(xq[:T])).cuda())
        torch.cuda.synchronize()
        assert model.profile_end()["input_gemm"]["launches"] == launches, T


@pytest.mark.parametrize("N,H,T", [(256, 200, (1 << 14) + 12), (128, 128, (1 << 14) + 60)])
def test_the_last_piece_of_a_long_sequence(orc, N, H, T):
    """Beyond 2^14 steps a layer runs in pieces.  The last one is short enough here for a launch that keeps the W x terms of all its
    steps in LDS, but it does not compute them: it needs the ring of the pieces before, beside tables that (256 cells) fill the LDS."""
    layers, x = wl.make_custom([16], N, H, LN | PROJ, 1, T, seed=23, weight_param=0.9 / N ** 0.5)
    model, _ = run_and_compare(orc, layers, x, f"rowlong{N}", trace=False)
    assert model.get_quant(0)["m_c"] <= 2  # three tables, none of them short


@pytest.mark.parametrize("H,flags,m_c,T,own", [
    (256, LN | PROJ | PH, 2, 12, 0), (256, LN | PROJ | CIFG, 1, 40, 0),  # no room for the form per row: four rows per workgroup
    (224, LN | PROJ, 2, 12, 0), (256, PROJ, 0, 16, 0), (256, LN | PROJ, 4, 12, 0),  # none for the terms of all steps
    (224, LN | PROJ, 2, 40, 0), (160, LN | PROJ, 2, 12, 1), (256, PROJ, 3, 16, 1), (256, LN | PROJ, 4, 8, 1),
])
def test_wide_projections_in_every_cell_format(orc, H, flags, m_c, T, own):
    """The tables of a cell format and a wide projection beside each other in LDS: whichever of the kernels without exchange has
    the room runs, with its own W x or the input matmul's."""
    import torch

    layers, x = wl.make_custom([48], 256, H, flags, 9, T, seed=H + m_c, weight_param=0.06)
    xd = calibrate_on_gpu(layers, x)
    layers[0].c_absmax = 0.9 * 2.0 ** m_c
    model, oracle = binding.prepare(layers), orc.prepare(layers)
    assert oracle.layer(0)["m_c"] == m_c
    xq = model.quantize_input(xd)
    model.set_option("spin_limit", 64)
    model.set_option("barrier_never_completes", 1)  # a kernel whose workgroups meet would give up
    model.profile_begin()
    y = model.forward(xq).cpu().numpy()
    launches = {k: v["launches"] for k, v in model.profile_end().items()}
    assert model.device_status() == 0 and launches["recurrent"] == 1 and launches["cell"] == 0
    assert launches["input_gemm"] == 1 - own
    assert_equal("y", y, np.asarray(orc.forward(oracle, xq.cpu().numpy())))


@pytest.mark.parametrize("B,T", [(5, 7), (5, 12), (70, 20)])
def test_two_directions_of_unlike_cell_formats(orc, B, T):
    """A format whose tables leave one direction no room for a workgroup per row: both run in one launch all the same."""
    import torch

    others = []
    layers, x = wl.make_custom([48], 256, 256, LN | PROJ, B, T, seed=5, weight_param=0.06)
    back, _ = wl.make_custom([48], 256, 256, LN | PROJ, B, T, seed=6, weight_param=0.06)
    xd = calibrate_on_gpu(layers, x)
    calibrate_on_gpu(back, x)
    layers[0].c_absmax = 0.9 * 2.0 ** 2
    for m_c in (2, 3):
        back[0].c_absmax = 0.9 * 2.0 ** m_c
        fwd, bwd = binding.prepare(layers), binding.prepare(back)
        bwd.set_option("reverse", 1)
        xq = fwd.quantize_input(xd)
        bwd.profile_begin()
        y = binding.forward_bidirectional(fwd, bwd, xq).cpu().numpy()
        others.append(bwd.profile_end()["other"]["launches"])
        assert fwd.device_status() == 0 and bwd.device_status() == 0
        xs = xq.cpu().numpy()
        assert_equal("forward", y[:, :, :256], np.asarray(orc.forward(orc.prepare(layers), xs)))
        assert_equal("backward", y[:, :, 256:], np.asarray(orc.forward(orc.prepare(back), xs, reverse=True)))
    assert others[0] == others[1], others  # a direction by itself has its input and its output turned around
