"""Which of the three ways a model of equal layers runs -- layer after layer, as one launch with a layer per XCD ("stack") or with a
workgroup per (layer, row) ("rows") -- at sizes where one way is well ahead and at some where it is close; all of them give the oracle's
integers."""
import numpy as np
import pytest

import lstm_workloads as wl
from parity_util import assert_equal, prepare_both, run_counted

pytestmark = pytest.mark.gpu
LN, PH, PROJ, CIFG = wl.LAYER_NORM, wl.PEEPHOLE, wl.PROJECTION, wl.CIFG


WAYS = {"layers": {"stack": 0, "row_stack": 0}, "stack": {"stack": 2, "row_stack": 0}, "rows": {"stack": 1, "row_stack": 2}}


@pytest.mark.parametrize("L,N,H,flags,B,T,chosen", [
    # us layer after layer, a layer per XCD, a workgroup per (layer, row) where it can run
    (8, 256, 256, LN, 64, 8, "stack"),       # 224, 194
    (2, 256, 256, LN, 4, 4, "rows"),         # 42, 45, 38
    (8, 128, 128, LN, 64, 8, "layers"),      # 133, 194
    (3, 1024, 1024, LN, 32, 64, "layers"),   # 705, 1080
    (3, 64, 64, 0, 32, 64, "rows"),          # 117, 341, 79
    (2, 512, 512, 0, 8, 16, "layers"),       # 76, 125
    (8, 1024, 256, LN | PROJ, 1, 1, "stack"),  # 162, 73
    (4, 320, 320, LN, 1000, 2, "layers"),    # 105, 647: the 32-row kernel
    (6, 64, 64, LN | PH, 12, 64, "rows"),    # 574, 589, 204
    (8, 48, 16, LN | PROJ, 2, 44, "layers"),  # 388, 429
    (3, 112, 32, PROJ, 13, 9, "rows"),       # 39, 92, 36
    (3, 80, 72, PH | PROJ, 44, 2, "rows"),   # 29, 64, 21
    (5, 192, 40, CIFG | LN | PROJ, 81, 5, "layers"),  # 78, 198
    (6, 128, 128, 0, 32, 48, "rows"),        # 220, 307, 106
    (8, 240, 240, LN, 1, 2, "stack"),        # 142, 69
    (7, 144, 28, LN | PROJ, 3, 1, "stack"),  # 72, 58
    (7, 188, 188, LN | PH, 31, 15, "stack"),  # 284, 204
])
def test_the_faster_way_is_taken(orc, L, N, H, flags, B, T, chosen):
    import torch

    layers, x = wl.make_custom([64] + [H] * (L - 1), N, H, flags, B, T, seed=L + N + B, weight_param=0.9 / N ** 0.5)
    model, oracle, xq = prepare_both(orc, layers, x)
    xd = torch.from_numpy(xq).cuda()
    y, n, way = run_counted(model, lambda: model.forward(xd).cpu().numpy())
    assert way == chosen and n["recurrent"] == (L if way == "layers" else 1), (way, n)
    can_run = {"layers": True, "stack": True, "rows": N <= 256 and L <= 6 and L * B <= 256}
    for other in WAYS:
        if other == chosen or not can_run[other]:
            continue
        for key, value in WAYS[other].items():
            model.set_option(key, value)
        y2, n, way = run_counted(model, lambda: model.forward(xd).cpu().numpy())
        assert way == other, (way, n)
        assert_equal("all ways", y, y2)
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
        y, n, way = run_counted(model, lambda: model.forward(xd[:T].contiguous()).cpu().numpy())
        assert way == ("stack" if stacked else "layers") and n["recurrent"] == (1 if stacked else 8), (T, way, n)
    ys = torch.empty(tuple(y.shape), dtype=torch.int8, device="cuda")
    model.forward_static(xd, ys)
    torch.cuda.synchronize()
    assert_equal("static", ys.cpu().numpy(), y)
    model.set_option("stack", 2)
    assert model.workspace_bytes(1000, 32) > limit
