"""The four-row recurrent kernel (small batches of layers with more than 256 cells): against the oracle at the edges of
its tiles, in long sequences against the groups of 16 rows, and its bounded waits."""
import numpy as np
import pytest

import lstm_workloads as wl
from parity_util import assert_equal, prepare_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("I,N,H,flags,B,T", [
    (20, 257, None, 0, 1, 6),  # five workgroups, the last with one cell
    (20, 300, None, wl.LAYER_NORM, 7, 20),  # a ragged group; tags of the statistics wrap at 16 steps
    (20, 400, None, wl.CIFG | wl.LAYER_NORM | wl.PEEPHOLE, 6, 5),
    (20, 512, None, wl.PEEPHOLE, 17, 4),
    (20, 520, None, wl.LAYER_NORM, 3, 4),  # k depth between two forms
    (20, 640, None, wl.CIFG, 4, 4),
    (20, 700, None, wl.LAYER_NORM | wl.PEEPHOLE, 5, 4),
    (20, 1024, None, wl.LAYER_NORM, 33, 3),
    (20, 321, 57, wl.LAYER_NORM | wl.PEEPHOLE | wl.PROJECTION, 9, 5),  # fewer projection tiles than workgroups
    (20, 1000, 999, wl.LAYER_NORM | wl.PROJECTION, 2, 3),  # four tiles to a workgroup
    (20, 2048, 640, wl.CIFG | wl.LAYER_NORM | wl.PROJECTION, 6, 3),  # a whole XCD per group
    (20, 330, 700, wl.LAYER_NORM | wl.PROJECTION, 5, 4),  # more outputs than its workgroups hold: another kernel
    (20, 2000, 130, wl.PEEPHOLE | wl.PROJECTION, 32, 3),  # every compute unit
])
def test_four_rows_per_group(orc, I, N, H, flags, B, T):
    """Two calls with carried state: y, h and c against the oracle."""
    import torch

    H = H or N
    layers, x = wl.make_custom([I], N, H, flags, B, T, seed=N + B, weight_param=0.9 / N ** 0.5)
    lib_model, orc_model, xq = prepare_both(orc, layers, x)
    want, tr = orc.forward(orc_model, xq, trace_layer=0)
    hs = torch.full((B * H,), lib_model.get_quant(0)["zp_h"], dtype=torch.int8).cuda()
    cs = torch.zeros(B * N, dtype=torch.int16).cuda()
    xd = torch.from_numpy(xq).cuda()
    for t0, t1 in ((0, 1), (1, T)):
        y = lib_model.forward(xd[t0:t1].contiguous(), h_state=hs, c_state=cs)
        torch.cuda.synchronize()
        assert lib_model.device_status() == 0
        assert_equal(f"y[{t0}:{t1}]", y.cpu().numpy(), want[t0:t1])
        assert_equal("h", hs.cpu().numpy().reshape(B, H), tr["h"][t1 - 1])
        assert_equal("c", cs.cpu().numpy().reshape(B, N), tr["c"][t1 - 1])


@pytest.mark.parametrize("flags", [0, wl.LAYER_NORM | wl.PEEPHOLE, wl.LAYER_NORM | wl.PROJECTION])
def test_long_sequence_matches_groups_of_16_rows(flags):
    """1100 steps (the tags of h and m wrap four times), every output."""
    import torch
    from paper_2101_05453_amd import binding

    layers, x = wl.make_custom([40], 512, 200 if flags & wl.PROJECTION else 512, flags, 30, 8, seed=5, weight_param=0.04)
    binding.calibrate(layers, torch.from_numpy(x).cuda())
    model = binding.prepare(layers)
    xq = torch.randint(-128, 128, (1100, 30, 40), dtype=torch.int8, device="cuda")
    y4 = model.forward(xq)
    model.set_option("rows16", 2)
    assert torch.equal(y4, model.forward(xq))
    assert model.device_status() == 0


@pytest.mark.parametrize("flags", [wl.LAYER_NORM, wl.LAYER_NORM | wl.PROJECTION])
def test_waits_give_up_and_the_model_recovers(flags):
    import torch
    from paper_2101_05453_amd import binding

    layers, x = wl.make_custom([40], 512, 512 if not flags & wl.PROJECTION else 100, flags, 8, 4, seed=6, weight_param=0.04)
    binding.calibrate(layers, torch.from_numpy(x).cuda())
    model = binding.prepare(layers)
    xq = torch.randint(-128, 128, (4, 8, 40), dtype=torch.int8, device="cuda")
    want = model.forward(xq).cpu()
    model.set_option("spin_limit", 64)
    model.set_option("barrier_never_completes", 1)
    model.forward(xq)
    torch.cuda.synchronize()
    assert model.device_status() == 1
    model.set_option("barrier_never_completes", 0)
    model.set_option("spin_limit", 1 << 21)
    model.set_option("reset_status", 1)
    assert torch.equal(model.forward(xq).cpu(), want)
    assert model.device_status() == 0
