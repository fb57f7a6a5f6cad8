"""Cells with six to eight integer bits: tanh is steep at zero and flat soon in those formats, and the kernels hold it in LDS
as the deltas and bases of that prefix only.  Cell states over the whole of their range go through it on every persistent
kernel, and the launches show that it was those that ran."""
import numpy as np
import pytest

import lstm_workloads as wl
from parity_util import assert_equal, calibrate_on_gpu

pytestmark = pytest.mark.gpu
LN, PH, PROJ, CIFG = wl.LAYER_NORM, wl.PEEPHOLE, wl.PROJECTION, wl.CIFG


@pytest.mark.parametrize("N,H,flags,B,options", [
    (64, 64, 0, 3, {"stack": 0}),                               # one workgroup per row
    (203, 203, LN | PH, 9, {"stack": 0, "rows16": 1}),          # the same, 16 waves
    (320, 320, LN | PH, 9, {"stack": 0, "rows16": 1}),          # groups of four rows over several workgroups
    (520, 130, CIFG | LN | PROJ, 30, {"stack": 0, "rows16": 1}),
    (320, 96, LN | PROJ, 21, {"stack": 0, "rows16": 2}),        # groups of 16 rows
    (512, 256, LN | PH | PROJ, 37, {"stack": 0, "rows16": 0}),  # groups of 32 rows
    (512, 256, LN | PH | PROJ, 37, {"stack": 2}),
    (320, 320, CIFG, 33, {"stack": 2}),
    (200, 200, LN, 37, {"stack": 0, "rows16": 0, "sparse": 2}),  # groups of 32 rows, R pruned two of four
    (512, 100, PH | PROJ, 40, {"stack": 0, "rows16": 0, "sparse": 2}),
])
@pytest.mark.parametrize("m_c", [6, 7, 8])
def test_wide_cell_formats(orc, N, H, flags, B, options, m_c):
    import torch

    from paper_2101_05453_amd import binding

    T = 4
    layers, x = wl.make_custom([48, H], N, H, flags, B, T, seed=N + m_c, weight_param=0.9 / N ** 0.5)
    if "sparse" in options:
        wl.prune_2of4(layers)
    xd = calibrate_on_gpu(layers, x)
    for s in layers:
        s.c_absmax = 2.0 ** m_c - 1
    model, oracle = binding.prepare(layers), orc.prepare(layers)
    assert all(oracle.layer(l)["m_c"] == m_c for l in range(2))
    for k, v in options.items():
        model.set_option(k, v)
    xq = model.quantize_input(xd)
    rng = np.random.default_rng(m_c)
    h0 = np.concatenate([np.full(B * H, oracle.layer(l)["zp_h"], np.int8) for l in range(2)])
    # every magnitude of the table: small ones on its steep part, then the whole int16 range with both ends
    c0 = rng.integers(-32768, 32768, 2 * B * N).astype(np.int16)
    c0[::2] = rng.integers(-4096, 4097, c0[::2].size)
    c0[:4] = [-32768, 32767, 1, -1]
    hs, cs = torch.from_numpy(h0.copy()).cuda(), torch.from_numpy(c0.copy()).cuda()
    model.profile_begin()
    y = model.forward(xq, h_state=hs, c_state=cs).cpu().numpy()
    launches = {k: v["launches"] for k, v in model.profile_end().items()}
    assert model.device_status() == 0
    # one launch per layer, or one for the stack; the path of one launch per step would have T per layer
    assert launches["recurrent"] == (1 if options["stack"] else 2) and launches["cell"] == 0, launches
    ho, co = h0.copy(), c0.copy()
    yo = orc.forward(oracle, xq.cpu().numpy(), h_state=ho, c_state=co)
    assert_equal("y", y, np.asarray(yo))
    assert_equal("h_state", hs.cpu().numpy(), ho)
    assert_equal("c_state", cs.cpu().numpy(), co)
