"""The SRU scan's rounds of four steps: step counts around whole rounds on every form of the scan (terms in tile order or
row-major, highway matrix or identity, either sigma table, the general form)."""
import numpy as np
import pytest

import lstm_workloads as wl
from test_gpu_sru import both, equal, quantize_x, sru, state_rows  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inputs,N,B", [
    ([64, 96], 96, 5),         # tile order: matrix, then identity
    ([64, 1284, 1284], 1284, 3),  # row-major: the general matmul's terms, small table
    ([1040, 1040], 1040, 330),  # row-major, the large table
    ([64], 512, 1030),         # tile order and matrix, more than one round of workgroups
    ([75, 37], 37, 4),         # cells not a multiple of four: the general form
])
def test_steps_around_whole_rounds(sru, inputs, N, B):  # noqa: F811
    import torch

    layers, x = wl.make_sru(inputs, N, B, 9, seed=N, weight_param=1.0 / N ** 0.5, input_param=1.5)
    sru.calibrate(layers, np.ascontiguousarray(x[:, :2]))
    lib_m, orc_m = both(sru, layers)
    xq = quantize_x(x, orc_m.get_quant(0))
    sel = np.array(sorted({0, 1, B // 2, B - 1}))
    c0 = np.random.default_rng(4).integers(-32768, 32768, size=B * N * len(layers)).astype(np.int16)
    for T in (1, 2, 3, 4, 5, 7, 8, 9):
        co = np.concatenate([r.ravel() for r in state_rows(c0, layers, B, sel)])
        yo, _ = orc_m.forward(np.ascontiguousarray(xq[:T, sel]), c_state=co, threads=8)
        cs = torch.from_numpy(c0.copy()).cuda()
        equal(f"y[{T}]", lib_m.forward(torch.from_numpy(np.ascontiguousarray(xq[:T])).cuda(), c_state=cs).cpu().numpy()[:, sel], yo)
        for g, w in zip(state_rows(cs.cpu().numpy(), layers, B, sel), state_rows(co, layers, len(sel), np.arange(len(sel)))):
            equal(f"c_state[{T}]", g, w)
