"""m in marked words (the 16-row and the 32-row kernel, tagged state with a projection; a stacked launch of one item per layer, whose layers
hand their rows on the same way): fewer steps than slots, slots that come round again, workgroups without outputs, rows beyond the
batch -- and values that look like the marks themselves."""
import numpy as np
import pytest
import torch

import lstm_workloads as wl
from paper_2101_05453_amd import binding
from parity_util import assert_equal, calibrate_on_gpu, run_and_compare

pytestmark = pytest.mark.gpu
LN, PH, PROJ, CIFG = wl.LAYER_NORM, wl.PEEPHOLE, wl.PROJECTION, wl.CIFG


@pytest.mark.parametrize("rows16", [0, 2])
@pytest.mark.parametrize("T", [1, 3, 5, 6, 13])
@pytest.mark.parametrize("N,H,B,flags", [
    (200, 152, 37, 0), (600, 296, 19, PH), (600, 200, 40, LN), (1100, 16, 33, LN | PH), (650, 640, 16, CIFG | LN | PH), (136, 24, 50, PH | CIFG),
])
def test_slots_in_turn(orc, N, H, B, flags, T, rows16):
    layers, x = wl.make_custom([24], N, H, flags | PROJ, B, T, seed=N + T, weight_param=0.9 / N ** 0.5)
    run_and_compare(orc, layers, x, f"m{N}h{H}t{T}", trace=False, options={"rows16": rows16})


@pytest.mark.parametrize("T", [3, 12])
@pytest.mark.parametrize("flags", [0, LN, PH | LN])
def test_two_directions(orc, flags, T):
    models, olds, x = [], [], None
    for seed in (3, 4):
        layers, xf = wl.make_custom([24], 300, 136, flags | PROJ, 21, T, seed=seed, weight_param=0.06)
        x = xf if x is None else x
        calibrate_on_gpu(layers, x)
        models.append(binding.prepare(layers))
        olds.append(orc.prepare(layers))
    models[1].set_option("reverse", 1)
    for m in models:
        m.set_option("rows16", 2)
    xq = models[0].quantize_input(torch.from_numpy(x).cuda())
    y = binding.forward_bidirectional(models[0], models[1], xq).cpu().numpy()
    assert all(m.device_status() == 0 for m in models)
    xh = xq.cpu().numpy()
    assert_equal("forward", y[:, :, :136], orc.forward(olds[0], xh))
    assert_equal("backward", y[:, :, 136:], orc.forward(olds[1], np.ascontiguousarray(xh[::-1]))[::-1])


def _ends_of_the_range(inputs, N, H, flags, B, T, most):
    """Cells driven to both ends of the range of m by turns, every eighth of them to either side of -127."""
    layers, x = wl.make_custom(inputs, N, H, flags, B, T, seed=1, weight_param=0.02)
    n = np.arange(N)
    for lay in layers:
        for g in (0, 1):  # input and forget gate open
            lay.b[g][:] = 5.0
        lay.b[2][:] = np.where(n % 2, 6.0, -6.0)
        lay.b[3][:] = np.where(n % 8 == 0, 2.5 + 2.0 * n / N, 6.0)
        if flags & LN:  # the biases alone
            for g in range(4):
                lay.Lw[g][:] = 0.05
    xd = calibrate_on_gpu(layers, x)
    for lay in layers:
        lay.m_min, lay.m_max = -most, most
        if not flags & PROJ:
            lay.h_min, lay.h_max = -most, most
    return layers, xd


def _words(m):  # of four cells, the first of eight
    m = np.ascontiguousarray(m[:, :, :m.shape[2] // 8 * 8])
    return m.view(np.uint32)[:, :, ::2]


@pytest.mark.parametrize("rows16", [0, 2])
@pytest.mark.parametrize("flags,most", [(0, 0.97), (PH | LN, 0.93)])
def test_values_that_look_like_marks(orc, flags, most, rows16):
    layers, xd = _ends_of_the_range([24], 200, 136, flags | PROJ, 37, 9, most)
    model, old = binding.prepare(layers), orc.prepare(layers)
    model.set_option("rows16", rows16)
    xq = model.quantize_input(xd)
    y = model.forward(xq)
    assert model.device_status() == 0
    want, trace = orc.forward(old, xq.cpu().numpy(), trace_layer=0)
    assert (_words(trace["m"]) == 0x7F807F80).any() and (_words(trace["m"]) == 0x7F807F81).any()
    assert_equal("y", y.cpu().numpy(), want)


@pytest.mark.parametrize("flags,most", [(0, 0.9), (PROJ, 0.97), (LN, 0.9), (PH | LN | PROJ, 0.93)])
@pytest.mark.parametrize("B", [1, 32])
def test_marks_between_layers_of_a_one_step_stack(orc, B, flags, most):
    T, L = 7, 3
    layers, xd = _ends_of_the_range([24] + [136 if flags & PROJ else 200] * (L - 1), 200, 136, flags, B, T, most)
    model, old = binding.prepare(layers), orc.prepare(layers)
    model.set_option("stack", 2)
    model.set_option("row_stack", 0)
    xq = model.quantize_input(xd)
    H = layers[0].output_size
    hs = torch.cat([torch.full((B * H,), model.get_quant(l)["zp_h"], dtype=torch.int8) for l in range(L)]).cuda()
    cs = torch.zeros(L * B * 200, dtype=torch.int16).cuda()
    y = torch.cat([model.forward(xq[t:t + 1].contiguous(), h_state=hs, c_state=cs) for t in range(T)])
    assert model.device_status() == 0
    want, trace = orc.forward(old, xq.cpu().numpy(), trace_layer=0)
    assert (_words(trace["m"]) == 0x7F807F80).any()
    assert_equal("y", y.cpu().numpy(), want)


@pytest.mark.parametrize("T", [1, 2, 3, 5, 6, 13])
@pytest.mark.parametrize("N,B,flags", [
    (650, 42, LN), (650, 43, LN),  # no room for the slots, and just enough
    (1024, 97, CIFG), (700, 70, PH | LN), (704, 65, 0), (1024, 500, CIFG | LN), (900, 511, PH | CIFG), (650, 301, PH),
])
def test_slots_of_the_state_in_turn(orc, N, B, flags, T):
    """The 32-row kernel at the longest k without a projection."""
    layers, x = wl.make_custom([24], N, N, flags, B, T, seed=N + T, weight_param=0.9 / N ** 0.5)
    rows = sorted({0, 31, 32, B // 2, B - 2, B - 1})
    run_and_compare(orc, layers, x, f"h{N}b{B}t{T}", trace=False, rows=rows, options={"rows16": 0})


@pytest.mark.parametrize("flags", [0, LN])
@pytest.mark.parametrize("N,B", [(700, 70), (1024, 300)])
@pytest.mark.parametrize("T", [3, 9])
def test_states_that_look_like_marks(orc, N, B, flags, T):
    layers, xd = _ends_of_the_range([24], N, N, flags, B, T, 0.9)
    model, old = binding.prepare(layers), orc.prepare(layers)
    model.set_option("rows16", 0)
    xq = model.quantize_input(xd)
    y = model.forward(xq)
    assert model.device_status() == 0
    rows = [0, 31, 32, 63, B // 2, B - 1]
    want, trace = orc.forward(old, np.ascontiguousarray(xq.cpu().numpy()[:, rows]), trace_layer=0)
    assert (_words(trace["m"])[:-1] == 0x7F807F80).any() and (_words(trace["m"])[:-1] == 0x7F807F81).any()
    assert_equal("y", y.cpu().numpy()[:, rows], want)


def test_waits_for_marked_state_give_up():
    N, B = 700, 70
    layers, x = wl.make_custom([24], N, N, LN, B, 5, seed=1, weight_param=0.03)
    calibrate_on_gpu(layers, x)
    m = binding.prepare(layers)
    m.set_option("rows16", 0)
    xq = m.quantize_input(torch.from_numpy(x).cuda())
    want = m.forward(xq)
    m.set_option("spin_limit", 64)
    m.set_option("barrier_never_completes", 1)
    m.forward(xq)
    assert m.device_status() == 1
    m.set_option("barrier_never_completes", 0)
    m.set_option("spin_limit", 1 << 21)
    m.set_option("reset_status", 1)
    assert torch.equal(m.forward(xq), want) and m.device_status() == 0


LONG = (1 << 14) + 9  # a launch takes 2^14 steps at most: the slots are marked again between two


@pytest.mark.parametrize("rows16", [0, 2])
@pytest.mark.parametrize("flags", [0, LN])
def test_slots_of_a_second_launch(orc, flags, rows16):
    layers, x = wl.make_custom([4], 136, 24, flags | PROJ, 35, LONG, seed=3, weight_param=0.08)
    run_and_compare(orc, layers, x, f"long{flags}", trace=False, rows=[0, 31, 34], options={"rows16": rows16})


@pytest.mark.parametrize("flags", [0, LN])
def test_slots_of_the_state_in_a_second_launch(flags):
    """The 32-row kernel at the longest k; against one launch per operation and step, which has no slots."""
    layers, x = wl.make_custom([4], 650, 650, flags, 43, LONG, seed=4, weight_param=0.04)
    calibrate_on_gpu(layers, np.ascontiguousarray(x[:64]))
    m = binding.prepare(layers)
    m.set_option("rows16", 0)
    xq = m.quantize_input(torch.from_numpy(x).cuda())
    y = m.forward(xq)
    assert m.device_status() == 0
    m.set_option("path", 1)
    assert torch.equal(m.forward(xq), y)
