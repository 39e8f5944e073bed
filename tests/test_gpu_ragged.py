"""GPU parity of the matrix-core step kernels where neither the streams nor the units fill whole
16 x 16 tiles: units are padded to quads, the last block of streams is short, and stream groups may
be unequal."""
import numpy as np
import pytest

import workloads as wl
from tests import test_gpu_window as tw
from tests.test_gpu_parity import run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,N", [([16], 9), ([21], 9), ([15, 17], 15), ([17, 31], 17), ([33], 31), ([30, 50], 33),
                                      ([250, 250], 20), ([131], 65), ([513], 18), ([1021], 12)])
def test_ragged_widths_and_streams_run_on_the_matrix_cores(layers, N):
    spec = wl.lstm_net(13, layers, 5)
    win, _ = run_both(wl.make_workload("ragged", spec, T=9, N=N, seed=71, scale=1.6 / max(layers) ** 0.5 / 4, bias_scale=0.2, masked_fraction=0.2),
                      label=f"ragged {layers}, N={N}")
    rec = [k for k in range(len(spec.nodes)) if win.g.step_build(k)[0] != "none"]
    assert rec and all(win.g.step_build(k, b)[0] == "matrix" for k in rec for b in (False, True))


@pytest.mark.parametrize("layers,N,builds", [([545], 4, ("matrix", "matrix")), ([513], 5, ("matrix", "matrix")), ([1021], 2, ("matrix", "matrix")),
                                             ([250], 8, ("matrix", "matrix")), ([290, 290], 3, ("matrix", "matrix")), ([290], 3, ("matrix", "wave"))])
def test_few_streams_where_the_register_build_needs_several_xcds(layers, N, builds):
    spec = wl.lstm_net(13, layers, 5)
    win, _ = run_both(wl.make_workload("few", spec, T=7, N=N, seed=72, scale=0.4 / max(layers) ** 0.5, bias_scale=0.2, masked_fraction=0.2),
                      label=f"{layers}, N={N}")
    rec = [k for k in range(len(spec.nodes)) if win.g.step_build(k)[0] != "none"]
    assert rec and all((win.g.step_build(k)[0], win.g.step_build(k, True)[0]) == builds for k in rec)


@pytest.mark.parametrize("env", [{"RNNG_MSTEP_LOCAL": "1"}, {"RNNG_MSTEP_LOCAL": "0"}, {"RNNG_MSTEP_LOCAL": "1", "RNNG_XCD_LOCAL": "0"},
                                 {"RNNG_MSTEP_LOCAL": "1", "RNNG_MSTEP_EW": "0"}, {"RNNG_MSTEP_LOCAL": "0", "RNNG_MSTEP_EW": "0", "RNNG_MSTEP_HOLD": "0"}])
@pytest.mark.parametrize("net,hidden,N", [("lstm", 3, 9), ("lstm", 18, 33), ("lstm", 250, 20), ("lstm", 384, 16), ("elman", 16, 9), ("elman", 512, 16), ("elman", 41, 140)])
def test_exchange_inside_and_across_xcds(monkeypatch, net, hidden, N, env):
    """One layer on the matrix cores: its stream groups each on an XCD (one to nine of them, several of an XCD's workgroups left over) or
    spread over all, written through or not, with wavefronts for the element-wise program alone or without."""
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    spec = wl.elman_net(7, hidden, 5) if net == "elman" else wl.lstm_net(7, [hidden], 5)
    win, _ = run_both(wl.make_workload("exchange", spec, T=21, N=N, seed=73, scale=0.4 / hidden ** 0.5, bias_scale=0.2, masked_fraction=0.2),
                      label=f"{net} {hidden}, N={N}, {env}")
    win.check()
    rec = [k for k in range(len(spec.nodes)) if win.g.step_build(k)[0] != "none"]
    assert rec and all(win.g.step_build(k, b)[0] == "matrix" for k in rec for b in (False, True))


@pytest.mark.parametrize("net,hidden,N", [("lstm", 3, 9), ("lstm", 18, 33), ("lstm", 250, 20), ("elman", 512, 16), ("elman", 41, 140), ("elman", 17, 500)])
def test_stream_groups_found_on_several_xcds(monkeypatch, net, hidden, N):
    """A launch that exchanges inside an XCD finds out that its groups do not share one, and writes through: the same bits, and no error."""
    spec = wl.elman_net(7, hidden, 5) if net == "elman" else wl.lstm_net(7, [hidden], 5)
    w = wl.make_workload("dealt", spec, T=21, N=N, seed=79, scale=0.4 / hidden ** 0.5, bias_scale=0.2, masked_fraction=0.2)
    wins = []
    for local in ("1", "2"):
        monkeypatch.setenv("RNNG_MSTEP_LOCAL", local)
        wins.append(run_both(w, label=f"{net} {hidden}, N={N}, RNNG_MSTEP_LOCAL={local}")[0])
    rec = [k for k in range(len(spec.nodes)) if wins[0].g.step_build(k)[0] != "none"]
    for k in rec:
        assert all(win.g.step_build(k, b)[0] == "matrix" for win in wins for b in (False, True))
        assert np.array_equal(wins[0].node_output(k), wins[1].node_output(k)) and np.array_equal(wins[0].node_state_grad(k), wins[1].node_state_grad(k))


@pytest.mark.parametrize("local", ["1", "2"])
@pytest.mark.parametrize("N", [20, 500])
def test_replayed_launches_find_out_about_their_xcds_anew(monkeypatch, local, N):
    """Captured backward passes, replayed: what the workgroups of a launch tell each other is cleared in every replay."""
    import torch
    monkeypatch.setenv("RNNG_MSTEP_LOCAL", local)
    spec = wl.lstm_net(7, [18], 5)
    w = wl.make_workload("replayed", spec, T=9, N=N, seed=80, scale=0.1, bias_scale=0.2, masked_fraction=0.2)
    win, _ = run_both(w, label=f"replayed, N={N}, RNNG_MSTEP_LOCAL={local}")
    rec = [k for k in range(len(spec.nodes)) if win.g.step_build(k)[0] != "none"]
    first = [win.node_state_grad(k) for k in rec]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        win.bptt()
    for _ in range(4):
        graph.replay()
        torch.cuda.synchronize()
        assert all(np.array_equal(a, win.node_state_grad(k)) for a, k in zip(first, rec))
        win.check()
        win.forward()
        win.bptt()


@pytest.mark.parametrize("env", [{}, {"RNNG_MSTEP_LOCAL": "0"}])
@pytest.mark.parametrize("layers,N", [([1], 9), ([3], 16), ([8], 64), ([17], 40), ([5, 9], 12)])
def test_small_layers_set_up_their_element_wise_wavefronts(monkeypatch, layers, N, env):
    """Layers whose weights are a load or two of a thread: the wavefronts for the element-wise program reach their items before the others have
    left anything behind.  The same bits in every window (a launch each), at other streams' values too."""
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    spec = wl.lstm_net(5, layers, 4)
    w = wl.make_workload("small", spec, T=3, N=N, seed=77, scale=0.5, bias_scale=0.2)
    win, _ = run_both(w, label=f"small {layers}, N={N}, {env}")
    rec = [k for k in range(len(spec.nodes)) if win.g.step_build(k)[0] != "none"]
    assert rec and all(win.g.step_build(k, b)[0] == "matrix" for k in rec for b in (False, True))
    (x,) = spec.input_nodes()
    first = [win.node_output(k) for k in rec] + [win.node_state_grad(k) for k in rec]
    other = {x: -w.inputs[x]}
    for _ in range(20):
        win.set_inputs(other)
        win.forward(); win.bptt()
        win.set_inputs(w.inputs)
        win.forward(); win.bptt()
        win.check()
        assert all(np.array_equal(a, b) for a, b in zip(first, [win.node_output(k) for k in rec] + [win.node_state_grad(k) for k in rec]))


@pytest.mark.parametrize("layers,N,T", [([3], 9, 1), ([16], 33, 7), ([64], 10, 8), ([65], 9, 9), ([70, 130], 14, 25), ([200], 70, 17)])
def test_element_wise_recurrences_at_many_streams(layers, N, T):
    """LSTM layers without output recurrence beyond the streams of the weights-in-registers build: units and streams that fill no wavefront,
    windows of fewer steps than are loaded ahead, at once and in pieces."""
    from paper_1503_02852_amd.runner import window_for
    spec = wl.lstm_net(7, layers, 5, output_recurrence=False)
    w = wl.make_workload("element_wise", spec, T=T, N=N, seed=75, scale=0.3, bias_scale=0.2, masked_fraction=0.2)
    win, _ = run_both(w, label=f"element-wise {layers}, N={N}")
    rec = [k for k in range(len(spec.nodes)) if win.g.step_build(k)[0] != "none"]
    assert rec and all(win.g.step_build(k, b) == ("wave", False) for k in rec for b in (False, True))
    pieces = window_for(w)
    for a, b in ((0, T // 3), (T // 3, T - 1), (T - 1, T)):
        if a < b:
            pieces.forward_range(a, b)
    pieces.check()
    assert all(np.array_equal(pieces.node_output(k), win.node_output(k)) for k in rec)


@pytest.mark.parametrize("window", ["1", "0"])
@pytest.mark.parametrize("layers,N", [([20], 1), ([65], 4), ([20], 5), ([70, 33], 8), ([33], 12)])
def test_element_wise_recurrences_in_every_form(monkeypatch, layers, N, window):
    """At few streams (backward below five on the lanes of the register build), tensors in one window or stored one by one, windows moved ahead."""
    monkeypatch.setenv("RNNG_STORE_WINDOW", window)
    spec = wl.lstm_net(8, layers, 4, output_recurrence=False)
    run_both(wl.make_workload("element_wise", spec, T=19, N=N, seed=81, scale=0.3, bias_scale=0.2, masked_fraction=0.2), label=f"element-wise {layers}, N={N}, RNNG_STORE_WINDOW={window}")
    monkeypatch.setitem(tw.WINDOW_NETS, "element_wise", lambda: (spec, N))
    tw.test_window_computed_in_pieces_equals_the_window_at_once("element_wise")
    tw.test_window_moved_ahead_with_carried_state("element_wise")


@pytest.mark.parametrize("env", [{"RNNG_MSTEP_EW": "0"}, {"RNNG_MSTEP_HOLD": "0"}, {"RNNG_MSTEP_HOLD": "20"}, {"RNNG_MSTEP_EW": "0", "RNNG_MSTEP_HOLD": "20"}])
@pytest.mark.parametrize("layers,N", [([128, 128], 16), ([40, 56], 35)])
def test_stacks_with_helper_members_without_wavefronts_of_their_own_or_held_back(monkeypatch, layers, N, env):
    for k, v in {**env, "RNNG_CHAIN_HELPERS": "1"}.items():
        monkeypatch.setenv(k, v)
    spec = wl.lstm_net(12, layers, 5)
    win, _ = run_both(wl.make_workload("stack", spec, T=17, N=N, seed=82, scale=0.4 / max(layers) ** 0.5, bias_scale=0.2, masked_fraction=0.2), label=f"stack {layers}, N={N}, {env}")
    rec = [k for k in range(len(spec.nodes)) if win.g.step_build(k)[0] != "none"]
    assert rec and all(win.g.step_build(k, b) == ("matrix", True) for k in rec for b in (False, True))
    assert all(win.g.step_build_has_helpers(k, True) for k in rec)


def saturated_tanh_net(dim):
    g = wl.GraphSpec()
    x = g.add_node(wl.INPUT, wl.LINEAR, dim, name="x")
    h = g.add_node(wl.ADD, wl.TANH, dim, name="h")
    out = g.add_node(wl.ADD, wl.LINEAR, dim, is_output=wl.SQUARED_ERROR, name="out")
    g.add_edge(x, h, wl.IDENTITY, 0); g.add_edge(h, h, wl.DIAG, 1); g.add_edge(h, out, wl.IDENTITY, 0)
    return g


@pytest.mark.parametrize("N", [1, 6, 40])
def test_derivative_of_a_saturated_tanh(N):
    """f'(s) = 1 - y^2 from the stored y, element by element: y^2 is not rounded before it is subtracted.  Of the window's last frame, whose
    error term is the output's alone, 1 - y^2 is rounded once and its product once: 2 x 2^-24 relative; a rounded square would cost 2^-25 / (1 - y^2)."""
    spec = saturated_tanh_net(37)
    w = wl.make_workload("saturated", spec, T=3, N=N, seed=78, scale=0.01)
    x, h, out = (spec.node_by_name(k) for k in ("x", "h", "out"))
    w.inputs[x][...] = np.sign(w.inputs[x]) * (3.0 + np.abs(w.inputs[x]) % 1.5)
    win, _ = run_both(w, label=f"saturated tanh, N={N}")
    assert win.g.step_build(h)[0] == "wave" and win.g.step_build(h, True)[0] == "wave"
    y = win.node_output(h)[-1].astype(np.float64)
    assert (1 - y * y).max() < 0.02
    expected = win.node_state_grad(out)[-1].astype(np.float64) * (1 - y * y)
    assert np.abs(win.node_state_grad(h)[-1] / expected - 1).max() < 2.1 * 2.0 ** -24


@pytest.mark.parametrize("N", [65535, 65536, 70000])
def test_element_wise_recurrences_beyond_16_bits_of_streams(N):
    """Every stream has a thread of its own, also where its number does not fit 16 bits."""
    spec = wl.lstm_net(2, [3], 2, output_recurrence=False)
    win, ref = run_both(wl.make_workload("element_wise", spec, T=3, N=N, seed=76, scale=0.3, bias_scale=0.2, masked_fraction=0.2), label=f"element-wise [3], N={N}")
    rec = [k for k in range(len(spec.nodes)) if win.g.step_build(k)[0] != "none"]
    assert rec and all(win.g.step_build(k, b) == ("wave", False) for k in rec for b in (False, True))
    for k in rec:      # the upper streams by themselves: a tensor's maximum need not lie among them
        assert np.abs(win.node_output(k)[:, 65530:] - ref["y"][k][:, 65530:]).max() < 1e-6
        assert np.abs(win.node_state_grad(k)[:, 65530:] + ref["delta"][k][:, 65530:]).max() < 1e-6


@pytest.mark.parametrize("net,hidden,N", [("lstm", 512, 16), ("lstm", 300, 40), ("elman", 1100, 33), ("elman", 2052, 9), ("elman", 132, 16), ("generalized", 260, 20)])
def test_streamed_weights_with_resident_chunks(monkeypatch, net, hidden, N):
    """Chunks of a source kept in registers and LDS: one to all but one of them, a ragged one among them, in one launch and in pieces."""
    monkeypatch.setenv("RNNG_STEP_BUILD", "stream")
    monkeypatch.setenv("RNNG_SMSTEP_RESIDENT", "1")
    from paper_1503_02852_amd.runner import window_for
    spec = {"lstm": lambda: wl.lstm_net(7, [hidden], 5), "elman": lambda: wl.elman_net(7, hidden, 5), "generalized": lambda: wl.generalized_net(8, hidden, 2, 4)}[net]()
    w = wl.make_workload("resident", spec, T=8, N=N, seed=74, scale=0.4 / hidden ** 0.5, bias_scale=0.2, masked_fraction=0.2)
    win, _ = run_both(w, label=f"resident {net} {hidden}, N={N}")
    rec = [k for k in range(len(spec.nodes)) if win.g.step_build(k)[0] != "none"]
    assert rec and all(win.g.step_build(k, b)[0] == "streaming" for k in rec for b in (False, True))
    pieces = window_for(w)
    for a, b in ((0, 1), (1, 4), (4, 8)):
        pieces.forward_range(a, b)
    pieces.check()
    assert all(np.array_equal(pieces.node_output(k), win.node_output(k)) for k in rec)


@pytest.mark.parametrize("N,T", [(3, 16400), (17, 8200)])
def test_long_windows_keep_their_step_kernel(N, T):
    """Tensors far below the 1 GiB that a step kernel addresses, with copies that 16-stream tiles
    whatever the stream count would have taken beyond it."""
    from paper_1503_02852_amd.runner import Window
    spec = wl.elman_net(8, 1024, 4)
    (x,), (o,) = spec.input_nodes(), spec.output_nodes()
    rng = np.random.default_rng(5)
    out = {}
    for frames in (T, 64):
        win = Window(spec.node_array(), spec.edge_array(), frames, N)
        if frames == T:
            weights = win.weights.clone().uniform_(-0.03, 0.03)
            inputs = rng.standard_normal((T, N, 8)).astype(np.float32)
        win.weights.copy_(weights)
        win.inputs[x] = win.weights.new_tensor(inputs[:frames])
        win.forward()
        win.check()
        assert win.g.step_build(1)[0] == "matrix"
        out[frames] = win.node_output(o)
    assert np.isfinite(out[T]).all() and np.allclose(out[T][:64], out[64], rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("layers,N", [([29, 21], 21), ([18], 9), ([513], 2), ([300], 7)])
def test_ragged_windows_in_pieces_and_moved_ahead(monkeypatch, layers, N):
    """History frames of the padded exchange tensors, in both window forms."""
    monkeypatch.setitem(tw.WINDOW_NETS, "ragged", lambda: (wl.lstm_net(8, layers, 4), N))
    if max(layers) > 100:      # (weights of 0.4 make a wide layer chaotic: 1e-7 in the inputs grows to 3e-5 in 24 frames of 513 units, at 0.07 it stays)
        make = wl.make_workload
        monkeypatch.setattr(wl, "make_workload", lambda *a, **k: make(*a, **{**k, "scale": 1.5 / max(layers) ** 0.5}))
    tw.test_window_computed_in_pieces_equals_the_window_at_once("ragged")
    tw.test_window_moved_ahead_with_carried_state("ragged")


@pytest.mark.parametrize("dim,T,N", [(4, 5, 1), (8, 9, 3), (36, 30, 7), (128, 3, 40), (6, 9, 3), (33, 9, 2)])
def test_element_wise_programs_of_ordinary_nodes(dim, T, N):
    """Programs over whole groups of four units and over others: products, maxima, every activation, biases, diagonal and
    identity connections, one of them delayed, against the oracle (bars of the parity tests)."""
    from tests.test_gpu_parity import run_both
    g = wl.GraphSpec()
    x = g.add_node(wl.INPUT, wl.LINEAR, dim, name="x")
    a = g.add_node(wl.ADD, wl.TANH, dim, has_bias=True, name="a")
    b = g.add_node(wl.ADD, wl.SIGMOID, dim, has_bias=True, name="b")
    m = g.add_node(wl.MUL, wl.LINEAR, dim, name="m")
    mx = g.add_node(wl.MAX, wl.LINEAR, dim, name="mx")
    r = g.add_node(wl.ADD, wl.RELU, dim, has_bias=True, name="r")
    o = g.add_node(wl.ADD, wl.SOFTMAX, 5, has_bias=True, is_output=wl.CROSS_ENTROPY, name="o")
    for src, dst, kind, delay in [(x, a, wl.FULL, 0), (x, b, wl.FULL, 0), (x, a, wl.DIAG, 1), (a, m, wl.IDENTITY, 0), (b, m, wl.DIAG, 0), (a, mx, wl.DIAG, 0),
                                  (b, mx, wl.IDENTITY, 1), (m, r, wl.DIAG, 0), (mx, r, wl.IDENTITY, 0), (a, r, wl.FULL, 0), (r, o, wl.FULL, 0)]:
        g.add_edge(src, dst, kind, delay)
    run_both(wl.make_workload("programs", g, T=T, N=N, seed=dim + T, scale=0.5, bias_scale=0.3), label=f"programs {dim}")
