"""The division of a step over eight waves, in the 32-row, the 16-row and the stacked kernel, at its edges: projections whose k steps
do not divide by eight (waves with fewer steps, or none), an odd number of outputs, one and two output tiles per workgroup
(partial sums through eight and through four slots of LDS), a second row tile, values beyond the part of the tables that LDS
holds, and the hand-off between the layers of a one-step stack."""
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
    (1850, 96, PROJ | LN, 40, 3),           # the same, the last wave with four
    (1024, 1024, LN, 70, 3),                # the deepest recurrent product
    (640, 600, PROJ | LN, 1000, 2),         # two row tiles, two output tiles
])
def test_division_over_the_waves(orc, N, H, flags, B, T):
    layers, x = wl.make_custom([48], N, H, flags, B, T, seed=N + H + B, weight_param=0.9 / N ** 0.5)
    rows = None if B <= 70 else [0, 31, 32, 63, 64, 500, 959, 960, B - 1]
    run_and_compare(orc, layers, x, f"waves{N}h{H}", trace=False, rows=rows, options={"rows16": 0})


@pytest.mark.parametrize("flags", [0, CIFG, PH, CIFG | PH, LN, LN | CIFG, LN | PH, LN | PH | CIFG])
@pytest.mark.parametrize("N,B,rows", [
    (1024, 513, [0, 31, 32, 63, 64, 511, 512]),             # a last group of one row: its second tile is empty
    (650, 1090, [0, 63, 545, 575, 576, 1023, 1024, 1089]),  # a second launch, of groups of 32
    (650, 1590, [0, 63, 1023, 1024, 1087, 1088, 1589]),     # a second launch, whose last tile is ragged
])
def test_two_row_tiles_at_the_deepest_k(orc, N, B, rows, flags):
    """Groups of 64 rows where R h is 1024 deep: every form without a projection."""
    layers, x = wl.make_custom([24], N, N, flags, B, 3, seed=N + B + flags, weight_param=0.9 / N ** 0.5)
    run_and_compare(orc, layers, x, f"two{N}b{B}f{flags}", trace=False, rows=rows, options={"rows16": 0})


@pytest.mark.parametrize("variant", range(8))  # coupled gates, peephole, layer norm
@pytest.mark.parametrize("N,H,B", [
    (60, 60, 33), (60, 40, 33), (60, 300, 20), (60, 700, 20),  # one workgroup per group: the state through the layer output
    (100, 400, 1500), (100, 700, 1200),  # two, and no room for the tagged words of all groups
    (200, 200, 40), (600, 600, 40), (700, 700, 21),  # tagged words
    (200, 150, 40), (600, 300, 40), (1100, 650, 21), (1100, 16, 21),  # with a projection; workgroups without outputs
])
def test_every_form_of_the_16_row_kernel(orc, N, H, B, variant):
    flags = variant | (PROJ if H != N else 0)
    layers, x = wl.make_custom([24], N, H, flags, B, 4, seed=N + H + variant, weight_param=0.9 / N ** 0.5)
    run_and_compare(orc, layers, x, f"r16_{N}_{H}_{flags}", trace=False, rows=None if B <= 40 else [0, 15, 16, 31, B // 2, B - 2, B - 1],
                    options={"rows16": 2})


@pytest.mark.parametrize("variant", range(8))
@pytest.mark.parametrize("N,H", [
    (60, 60), (200, 150), (600, 301), (700, 700), (1100, 700),  # the state through the layer output
    (200, 200), (600, 600), (200, 152), (600, 304), (1100, 16),  # tagged words
])
def test_every_form_of_the_32_row_kernel(orc, N, H, variant):
    flags = variant | (PROJ if H != N else 0)
    layers, x = wl.make_custom([24], N, H, flags, 37, 4, seed=N + H + variant, weight_param=0.9 / N ** 0.5)
    run_and_compare(orc, layers, x, f"r32_{N}_{H}_{flags}", trace=False, options={"rows16": 0})


@pytest.mark.parametrize("pruned", [0, 1])
@pytest.mark.parametrize("N,B,flags", [
    (1024, 1025, LN),            # one row is left
    (1024, 1536, 0),             # as many as one launch of groups of 32 holds
    (1024, 1537, CIFG | LN),     # one more: two tiles again
    (650, 1100, LN | PH), (650, 1500, CIFG),
])
def test_what_two_row_tiles_leave_over(orc, N, B, flags, pruned):
    """Rows beyond the last full launch of groups of 64 run in groups of 32 where one launch holds them, in the sparse form where
    the recurrent weights are 2:4."""
    layers, x = wl.make_custom([24], N, N, flags, B, 3, seed=N + B + flags, weight_param=0.9 / N ** 0.5)
    if pruned:
        wl.prune_2of4(layers)
    run_and_compare(orc, layers, x, f"rest{N}b{B}f{flags}", trace=False, rows=[0, 63, 1023, 1024, (1024 + B) // 2, B - 2, B - 1])


@pytest.mark.parametrize("N,H,flags,B,T", [
    (72, 9, PROJ, 5, 4),                    # two k steps of 64: most waves have none
    (300, 131, PROJ | LN, 20, 4),           # five k steps; odd outputs
    (1100, 33, PROJ | LN | PH, 17, 3),      # 18 k steps, three per wave: the last two waves have none
    (1024, 640, PROJ | LN, 37, 3),          # two output tiles of some workgroups
    (2048, 640, PROJ | LN | PH, 40, 3),     # four k steps per wave
    (2048, 640, PROJ | CIFG, 16, 3),
    (1024, 1024, LN | PH, 35, 3),           # the deepest recurrent product
    (1024, 1024, CIFG, 1, 3),
    (203, 203, LN, 21, 4),                  # the last piece of 16 cells of a row incomplete, rows of odd length
    (332, 332, 0, 33, 4),                   # the same, rows of a multiple of four
    (66, 66, LN | PH, 16, 4),               # a workgroup with two cells
])
def test_division_over_the_waves_of_16_rows(orc, N, H, flags, B, T):
    layers, x = wl.make_custom([48], N, H, flags, B, T, seed=N + H + B, weight_param=0.9 / N ** 0.5)
    run_and_compare(orc, layers, x, f"rows16_{N}h{H}", trace=False, options={"rows16": 2})


@pytest.mark.parametrize("N,H,flags,B,T", [
    (130, 130, 0, 20, 300),                  # the tags wrap at 256 steps; a last piece of eight cells with two
    (203, 203, LN, 21, 4),                   # rows of 208: the 16 cells of a lane end half way
    (332, 332, LN | PH, 33, 4),              # pairs straight from the lanes that make them
    (1024, 1024, CIFG, 128, 4),              # four pieces a thread, every compute unit
    (1100, 33, PROJ | PH, 17, 4),            # fewer pieces than threads: waves without any
    (700, 640, PROJ | LN, 40, 4),            # two and a half pieces a thread, two output tiles of some workgroups
    (128, 1000, PROJ | LN, 900, 3),          # no room for the words of so many groups: the counter
    (64, 64, LN, 20, 4),                     # one workgroup: nothing to exchange
])
def test_state_in_tagged_words(orc, N, H, flags, B, T):
    layers, x = wl.make_custom([40], N, H, flags, B, T, seed=N + H + T, weight_param=0.9 / N ** 0.5)
    rows = None if B <= 40 else [0, 15, 16, 17, B // 2, B - 1]
    run_and_compare(orc, layers, x, f"tags{N}h{H}", trace=False, rows=rows, options={"rows16": 2})


@pytest.mark.parametrize("N,H,flags,B,T", [
    (130, 16, PROJ, 40, 300),                # the tags wrap at 256 steps; one wave polls
    (200, 72, PROJ | LN, 33, 4),             # a second group of one row; the last pieces end within a wave
    (512, 256, PROJ | CIFG, 70, 4),          # two pieces a thread
    (700, 408, PROJ | LN | PH, 64, 4),       # three and four pieces
    (2048, 640, PROJ | LN, 300, 3),          # five; every compute unit, and a second launch
    (1024, 644, PROJ | LN, 40, 3),           # deeper, and no whole pieces: the counter
    (512, 100, PROJ, 40, 3),                 # no whole pieces
    (320, 416, PROJ, 40, 3),                 # more tiles of outputs than workgroups
    (130, 130, 0, 40, 300),                  # no projection: the tags wrap; a last piece of eight cells with two
    (203, 203, LN, 33, 4),                   # rows of 208
    (332, 332, LN | PH, 70, 4),
    (512, 512, CIFG, 600, 3),
    (640, 640, 0, 40, 5),                    # five pieces a thread
    (644, 644, LN, 40, 3),                   # deeper: the counter
])
def test_state_in_tagged_words_of_32_rows(orc, N, H, flags, B, T):
    layers, x = wl.make_custom([40], N, H, flags, B, T, seed=N + H + T, weight_param=0.9 / N ** 0.5)
    rows = None if B <= 40 else sorted({0, 31, 32, B // 2, B - 1})
    run_and_compare(orc, layers, x, f"tags32_{N}h{H}", trace=False, rows=rows, options={"rows16": 0})


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


@pytest.mark.parametrize("I,N,H,flags,B,T", [
    (64, 72, 9, PROJ, 5, 1),                 # one item per layer: the workgroups' own words; one of two has outputs
    (64, 300, 131, PROJ | LN, 32, 1),
    (128, 1024, 640, PROJ | LN, 9, 1),       # two output tiles of some workgroups, four slots
    (128, 640, 640, LN | PH, 32, 1),         # no projection: every workgroup stores rows
    (64, 72, 9, PROJ | CIFG, 37, 3),         # two row tiles: the first workgroup's word behind the barrier
    (64, 1100, 33, PROJ | LN | PH, 33, 2),
    (128, 1024, 640, PROJ | LN, 40, 2),
    (64, 1856, 96, PROJ | LN, 40, 2),        # eight k steps per wave, the last with four
    (64, 2048, 96, PROJ | LN, 9, 1),         # eight for all
])
def test_division_over_the_waves_of_a_stack(orc, I, N, H, flags, B, T):
    layers, x = wl.make_custom([I, H, H], N, H, flags, B, T, seed=N + H + B, weight_param=0.9 / N ** 0.5)
    run_and_compare(orc, layers, x, f"stack{N}h{H}", trace=False, options={"stack": 2})


@pytest.mark.parametrize("flags", [LN, PROJ | LN, 0])
def test_waits_of_a_one_step_stack_give_up(orc, flags):
    import torch

    H = 64 if flags & PROJ else 320
    layers, x = wl.make_custom([64, H, H], 320, H, flags, 7, 1, seed=11, weight_param=0.05)
    lib_model, orc_model, xq = prepare_both(orc, layers, x)
    lib_model.set_option("stack", 2)
    xd = torch.from_numpy(xq).cuda()
    lib_model.set_option("spin_limit", 64)
    lib_model.set_option("barrier_never_completes", 1)
    lib_model.forward(xd)
    torch.cuda.synchronize()
    assert lib_model.device_status() == 1
    lib_model.set_option("spin_limit", 1 << 21)
    lib_model.set_option("barrier_never_completes", 0)
    lib_model.set_option("reset_status", 1)
    assert_equal("recovered", lib_model.forward(xd).cpu().numpy(), np.asarray(orc.forward(orc_model, xq)))
    assert lib_model.device_status() == 0


@pytest.mark.parametrize("variant", [LN, LN | PH, LN | CIFG, LN | PH | CIFG])
@pytest.mark.parametrize("N,H,B,T", [
    (1792, 640, 37, 4),                        # 28 workgroups per group: adds
    (1793, 640, 37, 4), (1850, 24, 40, 5),     # 29: with a peephole statistics in words of each member
    (1920, 40, 33, 3), (1921, 40, 33, 3),      # 30, 31: without one too
    (2048, 640, 128, 3), (1990, 648, 33, 3),   # 32; too many outputs for it
    (2048, 16, 33, 70),                        # the tags come round
])
def test_statistics_of_wide_16_row_groups(orc, N, H, B, T, variant):
    layers, x = wl.make_custom([24], N, H, variant | PROJ, B, T, seed=N + H + variant, weight_param=0.9 / N ** 0.5)
    run_and_compare(orc, layers, x, f"s16_{N}_{H}_{variant}", trace=False, rows=[0, 15, 16, 31, B - 1], options={"rows16": 2})


@pytest.mark.parametrize("variant", [LN, LN | PH, LN | CIFG, LN | PH | CIFG])
@pytest.mark.parametrize("N,H,B", [(1921, 24, 21), (2048, 640, 33)])
def test_saturated_statistics_of_wide_16_row_groups(orc, N, H, B, variant):
    """A member's word holds its sum, its sum of squares and the step in 22, 36 and 6 bits: all of its 64 gate sums at either end of
    their range, where sum and squares come within 64 and within 2^22 of what the fields hold, in a row with members of both signs, in
    one of one sign (a variance of nearly 0), and beside ordinary members."""
    import torch

    layers, x = wl.make_custom([16], N, H, variant | PROJ, B, 5, seed=N + variant, weight_param=0.02)
    lay, member = layers[0], np.arange(N) // 64
    signs = {0: np.where(member % 2, 1.0, -1.0), 1: np.ones(N), 2: np.where(member < 5, 1.0, -1.0), 3: np.where(member % 3 == 0, 1.0, 0.0)}
    for g in range(1 if variant & CIFG else 0, 4):
        s = signs[g][:, None].astype(np.float32)
        lay.W[g] = np.ascontiguousarray(np.where(s != 0, s * (np.abs(lay.W[g]) + 0.05), lay.W[g] * 0.01).astype(np.float32))
        if variant & PH and g != 2:  # of the sign of the gate sum, where the state is of the sign of the z gate
            p = (0, 1, None, 2)[g]
            lay.P[p] = (np.abs(lay.P[p]) * np.where(signs[2] * signs[g] < 0, -1, 1)).astype(np.float32)
    x = np.ascontiguousarray((np.abs(x) + 0.3) * np.where(np.arange(B) % 2, 1.0, -1.0)[None, :, None]).astype(np.float32)
    lib_model, orc_model, xq = prepare_both(orc, layers, x, scale_x=60.0)
    lib_model.set_option("rows16", 2)
    y = lib_model.forward(torch.from_numpy(xq).cuda()).cpu().numpy()
    assert lib_model.device_status() == 0
    rows = [0, 1, 15, 16, B - 1]
    want, trace = orc.forward(orc_model, np.ascontiguousarray(xq[:, rows]), trace_layer=0)
    full = trace["g"][:, :, :, :N // 64 * 64].reshape(5, len(rows), 4, N // 64, 64)
    assert all((full[:, :, g] == v).all(axis=-1).any() for g in (1, 2, 3) for v in (32767, -32767))
    assert_equal("y", y[:, rows], np.asarray(want))
