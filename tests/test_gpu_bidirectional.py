"""lstm_int_forward_bidirectional: a forward stack and a backward stack (option "reverse") over the same input,
outputs side by side (Sec. 7: the bidirectional LSTM as two loops over the cell), against the oracle's two runs."""
import numpy as np
import pytest

import lstm_workloads as wl
from parity_util import assert_equal, calibrate_on_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    (0, [24], 40, 40, 5, 7),
    (wl.LAYER_NORM | wl.PROJECTION, [48, 24], 64, 24, 37, 6),
    (wl.CIFG | wl.LAYER_NORM | wl.PEEPHOLE, [64], 128, 128, 16, 9),
])
def test_bidirectional_outputs_side_by_side(orc, case, rows16=1):
    import torch
    from paper_2101_05453_amd import binding

    flags, inputs, N, H, B, T = case
    lay_f, x = wl.make_custom(inputs, N, H, flags, B, T, seed=31)
    lay_b, _ = wl.make_custom(inputs, N, H, flags, B, T, seed=77)  # the other direction has its own parameters
    xd = calibrate_on_gpu(lay_f, x)
    calibrate_on_gpu(lay_b, x)
    # the backward direction's statistics belong to the flipped sequence; the ranges of x are the same either way
    fwd, bwd = binding.prepare(lay_f, device=0), binding.prepare(lay_b, device=0)
    bwd.set_option("reverse", 1)
    for model in (fwd, bwd):
        model.set_option("rows16", rows16)
    of, ob = orc.prepare(lay_f), orc.prepare(lay_b)
    xq = fwd.quantize_input(xd)
    dims_f, dims_b = fwd.dims(), bwd.dims()
    rng = np.random.Generator(np.random.PCG64(3))
    st = {}
    for name, dims in (("f", dims_f), ("b", dims_b)):
        st[name] = (rng.integers(-128, 128, sum(B * d[2] for d in dims), dtype=np.int8),
                    rng.integers(-2000, 2000, sum(B * d[1] for d in dims), dtype=np.int16))
    dev = {k: (torch.from_numpy(v[0].copy()).cuda(), torch.from_numpy(v[1].copy()).cuda()) for k, v in st.items()}
    y = binding.forward_bidirectional(fwd, bwd, xq, state_fwd=dev["f"], state_bwd=dev["b"])
    torch.cuda.synchronize()
    assert fwd.device_status() == 0 and bwd.device_status() == 0
    xh = xq.cpu().numpy()
    hf, cf = st["f"][0].copy(), st["f"][1].copy()
    hb, cb = st["b"][0].copy(), st["b"][1].copy()
    yf = orc.forward(of, xh, h_state=hf, c_state=cf)
    yb = orc.forward(ob, xh, h_state=hb, c_state=cb, reverse=True)
    assert_equal("bidi.y", y.cpu().numpy(), np.concatenate([yf, yb], axis=2))
    for name, got, want in (("h_f", dev["f"][0], hf), ("c_f", dev["f"][1], cf), ("h_b", dev["b"][0], hb), ("c_b", dev["b"][1], cb)):
        assert_equal("bidi." + name, got.cpu().numpy(), want)
    # stateless call, caller-provided output and workspace
    ws = torch.empty(binding.bidirectional_workspace_bytes(fwd, bwd, T, B), dtype=torch.uint8, device="cuda")
    y2 = torch.full((T, B, dims_f[-1][2] + dims_b[-1][2]), 99, dtype=torch.int8, device="cuda")
    binding.forward_bidirectional(fwd, bwd, xq, y=y2, workspace=ws)
    torch.cuda.synchronize()
    assert_equal("bidi.y0", y2.cpu().numpy(), np.concatenate([orc.forward(of, xh), orc.forward(ob, xh, reverse=True)], axis=2))


@pytest.mark.parametrize("case", [
    (wl.PEEPHOLE, [30, 41], 41, 41, 3, 5),  # output rows that are no words of four
    (wl.LAYER_NORM | wl.PROJECTION, [64, 130], 320, 130, 70, 4),  # five groups per direction over the XCDs
    (wl.CIFG, [200], 512, 512, 33, 1),  # one step
    (wl.LAYER_NORM, [24], 1024, 1024, 128, 3),  # both directions fill the chip together
    (wl.LAYER_NORM, [24], 1024, 1024, 130, 2),  # one row more than fits: one after the other
])
def test_both_directions_in_one_launch(orc, case):
    test_bidirectional_outputs_side_by_side(orc, case)


@pytest.mark.parametrize("N", [130, 320, 650])  # the three k depths
@pytest.mark.parametrize("variant", range(8))
@pytest.mark.parametrize("proj", [0, 1])
def test_both_directions_in_one_launch_of_the_16_row_kernel(orc, proj, variant, N):
    """Every instantiation of the 16-row kernel that runs two directions side by side (CIFG, peephole, layer norm), with
    and without a projection, two groups per direction."""
    H = N - 5 if proj else N
    test_bidirectional_outputs_side_by_side(orc, (variant | (wl.PROJECTION if proj else 0), [24], N, H, 21, 4), rows16=2)


@pytest.mark.parametrize("N", [39, 128, 130, 256])  # four, eight and 16 waves; cells and outputs within a wave's block
@pytest.mark.parametrize("proj", [0, 1])
@pytest.mark.parametrize("variant", range(8))
@pytest.mark.parametrize("B", [6, 130])
def test_both_directions_in_one_launch_of_the_one_workgroup_kernel(orc, B, variant, proj, N):
    """Every instantiation of the kernels without exchange (CIFG, peephole, layer norm, projection) on both directions: a workgroup
    per row (6 rows), a workgroup per four rows, the last of each direction with two (130, beyond 256 rows of both together)."""
    H = N - 7 if proj else N
    test_bidirectional_outputs_side_by_side(orc, (variant | (wl.PROJECTION if proj else 0), [24], N, H, B, 4))


@pytest.mark.parametrize("N,T", [(64, 70), (39, 100), (128, 70), (250, 17), (250, 40)])
@pytest.mark.parametrize("flags", [0, wl.LAYER_NORM | wl.PEEPHOLE, wl.CIFG | wl.LAYER_NORM | wl.PROJECTION])
def test_both_directions_with_a_row_per_workgroup_from_the_input_matmul(orc, flags, N, T):
    """A workgroup per row where W x is not computed in its launch: the terms of both directions through the ring, the backward
    ones from the last step down; two layers, both ends' states."""
    H = N - 3 if flags & wl.PROJECTION else N
    test_bidirectional_outputs_side_by_side(orc, (flags, [24, H], N, H, 3, T))


@pytest.mark.parametrize("rows16", [1, 2])  # groups of four rows, of 16
def test_status_words_of_a_shared_launch(rows16):
    """Both directions in one launch: a misplaced workgroup (test hook) is reported by both models, a wait that gave up by
    the model of its direction alone, and the other direction's half of the output is right then."""
    import torch
    from paper_2101_05453_amd import binding

    _, x = wl.make_custom([24], 300, 300, wl.LAYER_NORM, 20, 5, seed=31)
    models = []
    for seed in (31, 77):
        layers, _ = wl.make_custom([24], 300, 300, wl.LAYER_NORM, 20, 5, seed=seed)
        xd = calibrate_on_gpu(layers, x)
        models.append(binding.prepare(layers, device=0))
        models[-1].set_option("rows16", rows16)
    fwd, bwd = models
    bwd.set_option("reverse", 1)
    xq = fwd.quantize_input(xd)
    want = binding.forward_bidirectional(fwd, bwd, xq)
    assert (fwd.device_status(), bwd.device_status()) == (0, 0)
    fwd.set_option("misplaced_workgroup", 1)
    binding.forward_bidirectional(fwd, bwd, xq)
    # 1: a wait that saw the 2 and gave up
    assert fwd.device_status() in (1, 2) and bwd.device_status() in (1, 2)
    fwd.set_option("misplaced_workgroup", 0)
    for m in models:
        m.set_option("reset_status", 1)
    bwd.set_option("spin_limit", 64)
    bwd.set_option("barrier_never_completes", 1)
    got = binding.forward_bidirectional(fwd, bwd, xq)
    assert (fwd.device_status(), bwd.device_status()) == (0, 1)
    assert torch.equal(got[:, :, :300], want[:, :, :300])
    bwd.set_option("spin_limit", 1 << 21)
    bwd.set_option("barrier_never_completes", 0)
    bwd.set_option("reset_status", 1)
    assert torch.equal(binding.forward_bidirectional(fwd, bwd, xq), want)
    assert (fwd.device_status(), bwd.device_status()) == (0, 0)


def test_bidirectional_argument_checks(orc):
    import torch
    from paper_2101_05453_amd import binding

    lay_f, x = wl.make_custom([24], 40, 40, 0, 3, 4, seed=1)
    lay_b, _ = wl.make_custom([24], 40, 40, 0, 3, 4, seed=2)
    xd = calibrate_on_gpu(lay_f, x)
    calibrate_on_gpu(lay_b, x)
    fwd, bwd = binding.prepare(lay_f, device=0), binding.prepare(lay_b, device=0)
    xq = fwd.quantize_input(xd)
    with pytest.raises(binding.LstmIntError) as e:  # the backward model must have "reverse" set
        binding.forward_bidirectional(fwd, bwd, xq)
    assert e.value.code == binding.E_INVALID_ARG
    bwd.set_option("reverse", 1)
    small = torch.empty(256, dtype=torch.uint8, device="cuda")
    with pytest.raises(binding.LstmIntError) as e:
        binding.forward_bidirectional(fwd, bwd, xq, workspace=small)
    assert e.value.code == binding.E_WORKSPACE
    lay_c, x2 = wl.make_custom([32], 40, 40, 0, 3, 4, seed=2)  # another input width
    calibrate_on_gpu(lay_c, x2)
    other = binding.prepare(lay_c, device=0)
    other.set_option("reverse", 1)
    with pytest.raises(binding.LstmIntError) as e:
        binding.forward_bidirectional(fwd, other, xq)
    assert e.value.code == binding.E_INVALID_ARG
    assert binding.forward_bidirectional(fwd, bwd, xq[:0]).shape == (0, 3, 80)
    torch.cuda.synchronize()
