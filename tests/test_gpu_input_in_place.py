"""The first layer's input term from x as the caller holds it: rows of 16-byte pieces in any batch are read in place, other
rows through a padded copy.  x ends where its buffer ends: the last block of 32 rows reaches beyond it."""
import numpy as np
import pytest

import lstm_workloads as wl
from parity_util import assert_equal, prepare_both
from test_gpu_gru import gru, run_both_paths  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("I,N,B,T,offset", [
    (16, 40, 1, 1, 0),
    (48, 64, 1, 40, 0),    # every block of 32 rows reaches beyond x
    (80, 96, 33, 3, 0),
    (272, 64, 5, 7, 0),    # k depth between two forms of the input GEMM
    (64, 320, 31, 3, 0),
    (1008, 70, 3, 5, 0),
    (48, 64, 37, 3, 8),    # x not on a 16-byte boundary: copied
    (24, 64, 37, 3, 0),    # rows of no whole pieces: copied
])
def test_lstm_reads_x_in_place(orc, I, N, B, T, offset):
    import torch

    layers, x = wl.make_custom([I], N, N, 0, B, T, seed=I + B, weight_param=0.9 / N ** 0.5)
    lib_model, orc_model, xq = prepare_both(orc, layers, x)
    want, _ = orc.forward(orc_model, xq, trace_layer=0)
    buf = torch.zeros(offset + xq.size, dtype=torch.int8, device="cuda")
    xd = buf[offset:].view(T, B, I)
    xd.copy_(torch.from_numpy(xq))
    assert_equal("y", lib_model.forward(xd).cpu().numpy(), want)
    assert lib_model.device_status() == 0


@pytest.mark.parametrize("inputs,N,B,T", [([48], 64, 1, 40), ([80], 96, 35, 3), ([24], 96, 35, 3)])
def test_gru_reads_x_in_place(gru, inputs, N, B, T):  # noqa: F811
    layers, x = wl.make_gru(inputs, N, B, T, seed=3, weight_param=0.9 / N ** 0.5, input_param=1.5)
    run_both_paths(gru, layers, x, f"gru{inputs}b{B}")


@pytest.mark.parametrize("I,N,B,T", [(48, 64, 1, 40), (96, 96, 35, 3), (24, 96, 35, 3)])
def test_sru_reads_x_in_place(I, N, B, T):
    import torch
    from oracle import sru as osru
    from paper_2101_05453_amd import binding

    layers, x = wl.make_sru([I], N, B, T, seed=4)
    osru.calibrate(layers, x, threads=4)
    m, om = binding.sru_prepare(layers, device=0), osru.SruModel(layers)
    q = om.get_quant(0)
    xq = np.clip(np.floor(x.astype(np.float64) / q["s_x"] + 0.5) + q["zp_x"], -128, 127).astype(np.int8)
    want, _ = om.forward(xq)
    assert_equal("y", m.forward(torch.from_numpy(xq).cuda()).cpu().numpy(), want)
