"""Layers of 129 to 256 cells in one workgroup of 16 waves, per row up to 256 rows and per four rows beyond: widths that end within
a wave's block of cells, leave waves without cells, or fill all of them; every combination of coupled gates, peephole and layer
norm; projections up to the workgroup's width; gate values beyond the part of the tables that LDS holds; a second layer, and rows
that are not a multiple of four."""
import numpy as np
import pytest

import lstm_workloads as wl
from parity_util import assert_equal, prepare_both, run_and_compare

pytestmark = pytest.mark.gpu
LN, PH, PROJ, CIFG = wl.LAYER_NORM, wl.PEEPHOLE, wl.PROJECTION, wl.CIFG


@pytest.mark.parametrize("flags", range(8))
@pytest.mark.parametrize("N,B,T", [(129, 1, 1), (144, 6, 4), (203, 5, 3), (256, 9, 4),
                                   (129, 257, 1), (144, 258, 4), (203, 261, 3), (256, 259, 4)])
def test_every_variant(orc, N, B, T, flags):
    layers, x = wl.make_custom([40, N], N, N, flags, B, T, seed=N + flags, weight_param=0.9 / N ** 0.5)
    run_and_compare(orc, layers, x, f"solo{N}f{flags}", trace=False, options={"stack": 0},
                    rows=None if B < 16 else [0, 3, 4, 127, 128, 255, B - 2, B - 1])


@pytest.mark.parametrize("N,H,flags", [
    (256, 256, PROJ | LN), (250, 17, PROJ | LN | PH), (131, 128, PROJ), (100, 200, PROJ | LN), (256, 241, PROJ | CIFG | PH),
])
@pytest.mark.parametrize("B", [7, 263])
def test_projections(orc, B, N, H, flags):
    layers, x = wl.make_custom([40], N, H, flags, B, 5, seed=N + H, weight_param=0.9 / N ** 0.5)
    run_and_compare(orc, layers, x, f"solo{N}h{H}", trace=False, rows=None if B < 16 else [0, 3, 4, 255, 256, B - 2, B - 1])


@pytest.mark.parametrize("flags", [0, LN, LN | PH, CIFG | LN])
def test_saturated_gates(orc, flags):
    import torch

    layers, x = wl.make_custom([64], 240, 240, flags, 1021, 4, seed=7 + flags, weight_param=0.3)
    lib_model, orc_model, xq = prepare_both(orc, layers, x, scale_x=60.0)
    y = lib_model.forward(torch.from_numpy(xq).cuda()).cpu().numpy()
    assert lib_model.device_status() == 0
    rows = [0, 3, 4, 511, 1019, 1020]
    assert_equal("y", y[:, rows], np.asarray(orc.forward(orc_model, np.ascontiguousarray(xq[:, rows]))))
