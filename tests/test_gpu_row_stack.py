"""Several layers of up to 256 cells in one launch, a workgroup per (layer, row): every variant in each of the three forms, pieces of the
sequence of every kind, layers of unlike widths, the first layer's W x from the input matmul and in the launch, carried state, both
directions, a wait that gives up, and the launch under capture; against the oracle and against layer after layer.  That it is this
launch that ran, the launches and the phase timers show."""
import numpy as np
import pytest

import lstm_workloads as wl
from paper_2101_05453_amd import binding
from parity_util import assert_equal, prepare_both, run_and_compare, run_counted

pytestmark = pytest.mark.gpu
LN, PH, PROJ, CIFG = wl.LAYER_NORM, wl.PEEPHOLE, wl.PROJECTION, wl.CIFG


def compare_rows(orc, layers, x, name, options):
    """run_and_compare on one launch of all layers."""
    import torch

    model, y = run_and_compare(orc, layers, x, name, trace=False, options=dict(options, row_stack=2))
    xd = torch.zeros(x.shape, dtype=torch.int8, device="cuda")
    _, n, way = run_counted(model, lambda: model.forward(xd))
    assert way == "rows" and n["recurrent"] == 1 and n["input_gemm"] <= 1, (n, way)
    return n


@pytest.mark.parametrize("flags", range(16))
@pytest.mark.parametrize("N", [40, 120, 250])
def test_every_variant(orc, N, flags):
    H = N - 9 if flags & PROJ else N
    layers, x = wl.make_custom([32, H, H], N, H, flags, 3, 21, seed=N + flags, weight_param=0.9 / N ** 0.5)
    compare_rows(orc, layers, x, f"rows{N}f{flags}", {})


@pytest.mark.parametrize("T,piece", [(1, 0), (2, 1), (7, 3), (16, 16), (17, 16), (33, 8), (40, 5)])
@pytest.mark.parametrize("I", [16, 75, 1024])
def test_pieces(orc, T, piece, I):
    """Pieces that end within a matrix product's 16 rows, at its last one and behind it; inputs in place, through the padded copy, and wide
    enough for the input matmul."""
    flags = (LN, 0, PH | LN, CIFG | LN | PROJ)[(T + I) % 4]
    N = (64, 100, 203)[T % 3]
    layers, x = wl.make_custom([I, N, N, N], N, N, flags, 5, T, seed=T + I, weight_param=0.9 / N ** 0.5)
    compare_rows(orc, layers, x, f"piece{T}.{piece}i{I}", {"row_stack_piece": piece})


@pytest.mark.parametrize("I,T,gemm", [(64, 12, 0), (64, 200, 0), (1024, 12, 1), (1024, 200, 1)])
def test_the_first_layers_input(orc, I, T, gemm):
    """W x of the first layer in the launch or by the input matmul."""
    layers, x = wl.make_custom([I, 256], 256, 256, 0, 30, T, seed=I + T, weight_param=0.05)
    assert compare_rows(orc, layers, x, f"first{I}.{T}", {})["input_gemm"] == gemm


@pytest.mark.parametrize("L,N,B,T,flags,rows", [(6, 96, 42, 12, LN, True), (2, 128, 128, 5, 0, True), (2, 128, 129, 5, 0, False),
                                                (7, 64, 4, 9, 0, False), (2, 257, 2, 9, 0, False)])
def test_limits(orc, L, N, B, T, flags, rows):
    """As many rows as there are compute units, and one more; as many layers as the arguments hold; cells beyond the forms."""
    import torch

    layers, x = wl.make_custom([64] + [N] * (L - 1), N, N, flags, B, T, seed=L + N, weight_param=0.9 / N ** 0.5)
    model, oracle, xq = prepare_both(orc, layers, x)
    xd = torch.from_numpy(xq).cuda()
    model.set_option("row_stack", 2)
    model.set_option("stack_step_ns", 1000000)  # (the launch of a layer per XCD is never the faster way)
    y, n, way = run_counted(model, lambda: model.forward(xd).cpu().numpy())
    assert way == ("rows" if rows else "layers") and n["recurrent"] == (1 if rows else L), (n, way)
    model.set_option("row_stack", 0)
    model.set_option("stack", 0)
    other, n, way = run_counted(model, lambda: model.forward(xd).cpu().numpy())
    assert way == "layers" and n["recurrent"] == L, (n, way)
    assert_equal("both ways", y, other)
    at = sorted({0, B // 2, B - 1})
    assert_equal("y", y[:, at], np.asarray(orc.forward(oracle, np.ascontiguousarray(xq[:, at]))))


@pytest.mark.parametrize("reverse", [0, 1])
def test_carried_state(orc, reverse):
    """A sequence in three calls against one call, state of every layer among it; the other direction of time too."""
    import torch

    T, B, N = 23, 6, 72
    layers, x = wl.make_custom([40, N, N], N, N, LN, B, T, seed=11, weight_param=0.1)
    model, oracle, xq = prepare_both(orc, layers, x)
    xd = torch.from_numpy(xq).cuda()
    model.set_option("reverse", reverse)
    got = {}
    for way in (2, 0):
        model.set_option("row_stack", way)
        model.set_option("stack", 1 if way else 0)
        h = torch.cat([torch.full((B * N,), model.get_quant(l)["zp_h"], dtype=torch.int8, device="cuda") for l in range(3)])
        c = torch.zeros(3 * B * N, dtype=torch.int16, device="cuda")
        cuts = [(0, 9), (9, 10), (10, T)]
        ys = []
        for a, b in cuts[::-1] if reverse else cuts:
            y, _, ran = run_counted(model, lambda: model.forward(xd[a:b].contiguous(), h_state=h, c_state=c))
            assert ran == ("rows" if way else "layers")
            ys.append(y)
        got[way] = [torch.cat(ys[::-1] if reverse else ys).cpu().numpy(), h.cpu().numpy(), c.cpu().numpy()]
    assert model.device_status() == 0
    for name, a, b in zip("yhc", got[2], got[0]):
        assert_equal(name, a, b)
    assert_equal("oracle", got[2][0], np.asarray(orc.forward(oracle, xq, reverse=bool(reverse))))


@pytest.mark.parametrize("N,I,B,T,flags", [(60, 40, 5, 19, LN), (64, 1024, 30, 34, 0), (200, 64, 3, 18, LN | PH), (96, 50, 1, 1, LN | PROJ)])
def test_two_directions(orc, N, I, B, T, flags):
    import torch

    H = N - 12 if flags & PROJ else N
    layers, x = wl.make_custom([I, H, H], N, H, flags, B, T, seed=5, weight_param=0.9 / N ** 0.5)
    back, _ = wl.make_custom([I, H, H], N, H, flags, B, T, seed=6, weight_param=0.9 / N ** 0.5)
    fwd, ofwd, xq = prepare_both(orc, layers, x)
    for a, b in zip(back, layers):
        a.x_min, a.x_max = b.x_min, b.x_max
    from parity_util import calibrate_on_gpu

    calibrate_on_gpu(back, x)
    back[0].x_min, back[0].x_max = layers[0].x_min, layers[0].x_max
    bwd, obwd = binding.prepare(back), orc.prepare(back)
    bwd.set_option("reverse", 1)
    xd = torch.from_numpy(xq).cuda()
    ys = []
    for way in (2, 0):
        fwd.set_option("row_stack", way)
        states = [(torch.zeros(3 * B * H, dtype=torch.int8, device="cuda"), torch.zeros(3 * B * N, dtype=torch.int16, device="cuda")) for _ in range(2)]
        bwd.profile_begin()
        y, n, ran = run_counted(fwd, lambda: binding.forward_bidirectional(fwd, bwd, xd, state_fwd=states[0], state_bwd=states[1]))
        # one launch, in the profiles of both models; else one for each layer of either direction or of both
        assert ran == ("rows" if way else "layers") and bwd.profile_end()["recurrent"]["launches"] == n["recurrent"] == (1 if way else 3), n
        ys.append([y.cpu().numpy()] + [s.cpu().numpy() for p in states for s in p])
    assert fwd.device_status() == 0 and bwd.device_status() == 0
    for a, b in zip(*ys):
        assert_equal("both ways", a, b)
    fwd.set_option("row_stack", 2)
    y = binding.forward_bidirectional(fwd, bwd, xd).cpu().numpy()
    assert_equal("forward", y[:, :, :H], np.asarray(orc.forward(ofwd, xq)))
    assert_equal("backward", y[:, :, H:], np.asarray(orc.forward(obwd, xq, reverse=True)))


def test_layers_of_unlike_widths(orc):
    """Narrow layers beside wide ones in the form of the widest."""
    a, x = wl.make_custom([48], 200, 200, LN, 4, 20, seed=2, weight_param=0.07)
    b, _ = wl.make_custom([200], 40, 40, LN, 4, 20, seed=3, weight_param=0.1)
    c, _ = wl.make_custom([40], 130, 130, LN, 4, 20, seed=4, weight_param=0.08)
    compare_rows(orc, a + b + c, x, "unlike", {})


def test_a_wait_that_gives_up(orc):
    import torch

    layers, x = wl.make_custom([64, 64], 64, 64, 0, 4, 40, seed=9, weight_param=0.1)
    model, oracle, xq = prepare_both(orc, layers, x)
    xd = torch.from_numpy(xq).cuda()
    model.set_option("row_stack", 2)
    model.set_option("spin_limit", 16)
    model.set_option("barrier_never_completes", 1)
    model.forward(xd)
    torch.cuda.synchronize()
    assert model.device_status() != 0
    for key, value in (("barrier_never_completes", 0), ("spin_limit", 1 << 21), ("reset_status", 1)):
        model.set_option(key, value)
    assert_equal("y", model.forward(xd).cpu().numpy(), np.asarray(orc.forward(oracle, xq)))
    assert model.device_status() == 0


@pytest.mark.parametrize("cooperative", [0, 1])
def test_several_streams(orc, cooperative):
    """Launches of all sizes on eight streams at once: more workgroups than compute units."""
    import torch

    models, inputs, want = [], [], []
    for i, (L, N, B, T) in enumerate([(6, 64, 42, 40), (2, 200, 128, 20), (3, 96, 7, 64), (4, 130, 5, 50)]):
        layers, x = wl.make_custom([48] + [N] * (L - 1), N, N, LN if i % 2 else 0, B, T, seed=i, weight_param=0.9 / N ** 0.5)
        model, oracle, xq = prepare_both(orc, layers, x)
        model.set_option("row_stack", 2)
        model.set_option("cooperative_launch", cooperative)
        models.append(model)
        inputs.append(torch.from_numpy(xq).cuda())
        assert run_counted(model, lambda: model.forward(inputs[-1]))[2] == "rows"
        rows = sorted({0, B - 1})
        want.append((rows, np.asarray(orc.forward(oracle, np.ascontiguousarray(xq[:, rows])))))
    streams = [torch.cuda.Stream() for _ in range(8)]
    spaces = [torch.empty(models[i % 4].workspace_bytes(*inputs[i % 4].shape[:2]), dtype=torch.uint8, device="cuda") for i in range(8)]
    got = [[] for _ in range(8)]
    torch.cuda.synchronize()
    for _ in range(3):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                got[i].append(models[i % 4].forward(inputs[i % 4], workspace=spaces[i]))
    torch.cuda.synchronize()
    assert all(m.device_status() == 0 for m in models)
    for i, ys in enumerate(got):
        rows, y = want[i % 4]
        assert_equal("oracle", ys[0].cpu().numpy()[:, rows], y)
        for other in ys[1:] + got[i % 4]:
            assert_equal("every call", other.cpu().numpy(), ys[0].cpu().numpy())


@pytest.mark.parametrize("I", [64, 1024])
def test_captured_in_a_hip_graph(orc, I):
    import torch

    layers, x = wl.make_custom([I, 96, 96], 96, 96, LN, 6, 30, seed=13, weight_param=0.09)
    model, oracle, xq = prepare_both(orc, layers, x)
    model.set_option("row_stack", 2)
    inputs = [xq, np.ascontiguousarray(xq[::-1]), np.ascontiguousarray(xq[:, ::-1])]
    xd = torch.from_numpy(xq).cuda()
    ws = torch.empty(model.workspace_bytes(30, 6), dtype=torch.uint8, device="cuda")
    y = torch.empty((30, 6, 96), dtype=torch.int8, device="cuda")
    assert run_counted(model, lambda: model.forward(xd, y=y, workspace=ws))[2] == "rows"
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        model.forward(xd, y=y, workspace=ws)
    for xi in inputs:
        xd.copy_(torch.from_numpy(xi))
        ws.random_(0, 255)
        graph.replay()
        torch.cuda.synchronize()
        assert_equal("replay", y.cpu().numpy(), np.asarray(orc.forward(oracle, xi)))
    assert model.device_status() == 0
