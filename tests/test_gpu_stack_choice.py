"""Which of the two ways a model of equal layers runs, layer after layer or as one stacked launch, by the number of launches, at
sizes where one way is well ahead and at some where it is close; both ways give the oracle's integers."""
import numpy as np
import pytest

import lstm_workloads as wl
from parity_util import assert_equal, prepare_both

pytestmark = pytest.mark.gpu
LN, PH, PROJ, CIFG = wl.LAYER_NORM, wl.PEEPHOLE, wl.PROJECTION, wl.CIFG


def forward_counted(model, xd):
    import torch

    model.profile_begin()
    y = model.forward(xd)
    torch.cuda.synchronize()
    assert model.device_status() == 0
    return y.cpu().numpy(), model.profile_end()["recurrent"]["launches"]


@pytest.mark.parametrize("L,N,H,flags,B,T,stacked", [
    # us stacked, one after the other
    (8, 256, 256, LN, 64, 8, True),       # 193, 232
    (2, 256, 256, LN, 4, 4, False),       # 45, 42
    (8, 128, 128, LN, 64, 8, False),      # 192, 143
    (3, 1024, 1024, LN, 32, 64, False),   # 1050, 707
    (3, 64, 64, 0, 32, 64, False),        # 335, 117
    (2, 512, 512, 0, 8, 16, False),       # 125, 76
    (8, 1024, 256, LN | PROJ, 1, 1, True),  # 81, 163
    (4, 320, 320, LN, 1000, 2, False),    # 640, 106: the 32-row kernel
    (6, 64, 64, LN | PH, 12, 64, False),  # 591, 583
    (8, 48, 16, LN | PROJ, 2, 44, False),  # 430, 414
    (3, 112, 32, PROJ, 13, 9, False),     # 91, 42
    (3, 80, 72, PH | PROJ, 44, 2, False),  # 66, 31
    (5, 192, 40, CIFG | LN | PROJ, 81, 5, False),  # 197, 94
    (6, 128, 128, 0, 32, 48, False),      # 304, 223
    (8, 240, 240, LN, 1, 2, True),        # 69, 143
    (7, 144, 28, LN | PROJ, 3, 1, True),  # 65, 90
    (7, 188, 188, LN | PH, 31, 15, True),  # 204, 306
])
def test_the_faster_way_is_taken(orc, L, N, H, flags, B, T, stacked):
    import torch

    layers, x = wl.make_custom([64] + [H] * (L - 1), N, H, flags, B, T, seed=L + N + B, weight_param=0.9 / N ** 0.5)
    model, oracle, xq = prepare_both(orc, layers, x)
    xd = torch.from_numpy(xq).cuda()
    y, launches = forward_counted(model, xd)
    assert launches == (1 if stacked else L), launches
    model.set_option("stack", 0 if stacked else 2)
    other, launches = forward_counted(model, xd)
    assert launches == (L if stacked else 1), launches
    assert_equal("both ways", y, other)
    rows = list(range(min(B, 4))) + [B - 1]
    assert_equal("y", y[:, rows], np.asarray(orc.forward(oracle, np.ascontiguousarray(xq[:, rows]))))


def test_the_choice_keeps_to_the_static_workspace(orc):
    """A call whose layers fit the library's own workspace one after the other, but not as a stack, runs them one after the
    other however short a stacked item is said to be."""
    import torch

    layers, x = wl.make_custom([64] + [64] * 7, 64, 64, 0, 32, 4, seed=3, weight_param=0.1)
    model, oracle, xq = prepare_both(orc, layers, x)
    model.set_option("stack_step_ns", 1)
    xd = torch.from_numpy(np.concatenate([xq] * 250)).cuda()
    limit = 32 << 20
    for T, stacked in ((700, True), (1000, False)):
        assert model.workspace_bytes(T, 32) <= limit
        y, launches = forward_counted(model, xd[:T].contiguous())
        assert launches == (1 if stacked else 8), (T, launches)
    ys = torch.empty(tuple(y.shape), dtype=torch.int8, device="cuda")
    model.forward_static(xd, ys)
    torch.cuda.synchronize()
    assert_equal("static", ys.cpu().numpy(), y)
    model.set_option("stack", 2)
    assert model.workspace_bytes(1000, 32) > limit
