"""The 32-row kernel's division of a step over eight waves, at its edges: projections whose k steps do not divide by eight
(waves with fewer steps, or none), an odd number of outputs, one and two output tiles per workgroup (partial sums through
eight and through four slots of LDS), a second row tile, and values beyond the part of the tables that LDS holds."""
import numpy as np
import pytest

import lstm_workloads as wl
from parity_util import assert_equal, prepare_both, run_and_compare

pytestmark = pytest.mark.gpu
LN, PH, PROJ, CIFG = wl.LAYER_NORM, wl.PEEPHOLE, wl.PROJECTION, wl.CIFG


@pytest.mark.parametrize("N,H,flags,B,T", [
    (72, 9, PROJ, 5, 4),                    # 4 k steps: half of the waves have none
    (300, 131, PROJ | LN, 40, 4),           # 12 k steps, two per wave: the last two waves have none; odd outputs
    (1100, 33, PROJ | LN | PH, 33, 3),      # 36 k steps, five per wave: the last wave has one
    (1024, 640, PROJ | LN, 37, 3),          # two output tiles of some workgroups, four slots
    (640, 640, PROJ | CIFG, 64, 3),         # the same at another width
    (2048, 640, PROJ | LN | PH, 40, 3),     # eight k steps per wave
    (1024, 1024, LN, 70, 3),                # the deepest recurrent product
    (640, 600, PROJ | LN, 1000, 2),         # two row tiles, two output tiles
])
def test_division_over_the_waves(orc, N, H, flags, B, T):
    layers, x = wl.make_custom([48], N, H, flags, B, T, seed=N + H + B, weight_param=0.9 / N ** 0.5)
    rows = None if B <= 70 else [0, 31, 32, 63, 64, 500, 959, 960, B - 1]
    run_and_compare(orc, layers, x, f"waves{N}h{H}", trace=False, rows=rows, options={"rows16": 0})


@pytest.mark.parametrize("N,H,flags", [
    (320, 320, 0), (320, 320, LN | PH),  # the tables whole in LDS
    (1024, 640, LN | PROJ),              # W_proj leaves no room for that: lookups beyond the prefix
])
def test_saturated_gates(orc, N, H, flags):
    """Features 60 times as large as those the statistics are from drive the gates to both ends of the tables."""
    import torch

    layers, x = wl.make_custom([64], N, H, flags, 33, 4, seed=5 + N, weight_param=0.3 if N < 1024 else 0.1)
    lib_model, orc_model, xq = prepare_both(orc, layers, x, scale_x=60.0)
    lib_model.set_option("rows16", 0)
    y = lib_model.forward(torch.from_numpy(xq).cuda()).cpu().numpy()
    assert lib_model.device_status() == 0
    assert_equal("y", y, np.asarray(orc.forward(orc_model, xq)))
