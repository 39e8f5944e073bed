"""rnn_forward_static (the entry point for callers that cannot allocate device memory: its
workspace is a device array inside the library) against rnn_forward on a workspace of the
caller's, through the C ABI: same kernels, so the output layers' activations must agree to the
forward bar (1e-4 normwise; in fact to the last bit), on two calls in a row, the second with a
smaller window, which must not see what the first left in the shared array."""
import numpy as np
import pytest

import workloads as wl
from oracle import graph_oracle as go

pytestmark = pytest.mark.gpu

OUT_TOL = 1e-4


def nerr(a, b):
    den = np.abs(b).max()
    return np.abs(np.asarray(a, np.float64) - b).max() / den if den > 0 else np.abs(a).max()


def outputs_both_ways(w):
    import torch
    from paper_1503_02852_amd.runner import window_for
    win = window_for(w)
    win.forward()                      # caller's workspace; also loads the kernels
    ref = {k: win.node_output(k).copy() for k in w.spec.output_nodes()}
    outs = {k: torch.full((w.T, w.N, w.spec.nodes[k]["dim"]), float("nan"), dtype=torch.float32, device=win.dev)
            for k in w.spec.output_nodes()}
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    win.g.forward_static(win.weights.data_ptr(), win._input_ptrs(), [outs[k].data_ptr() for k in w.spec.output_nodes()],
                         w.T, w.N, win._stream())
    win.check()
    assert torch.cuda.memory_allocated() == before
    got = {k: v.cpu().numpy() for k, v in outs.items()}
    return win, ref, got


@pytest.mark.parametrize("spec_fn", [lambda: wl.lstm_net(10, [48, 40], 6), lambda: wl.generalized_net(8, 32, 2, 5)])
def test_static_workspace_forward_equals_forward_two_calls_in_a_row(spec_fn):
    spec = spec_fn()
    for T, N, seed in ((40, 3, 71), (9, 2, 72)):          # the second window is smaller
        w = wl.make_workload("static", spec, T=T, N=N, seed=seed, scale=0.4, bias_scale=0.3)
        print(f"[static] T={T} N={N} nodes={len(spec.nodes)}", flush=True)
        win, ref, got = outputs_both_ways(w)
        y, _ = go.forward(spec.nodes, spec.edges, w.weights, w.biases, w.inputs, T, N)
        for k in spec.output_nodes():
            assert nerr(got[k], ref[k].astype(np.float64)) < OUT_TOL
            assert np.array_equal(got[k], ref[k])
            assert nerr(got[k], y[k]) < OUT_TOL
        # the handle's window now lives in the static array: the backward pass works on it
        win.bptt()
        loss = win.compute_grads(want_loss=True)
        full = go.forward_bptt(spec.nodes, spec.edges, w.weights, w.biases, w.inputs, w.targets, T, N)
        assert abs(loss - full["loss"]) <= 1e-5 * max(1.0, abs(full["loss"]))
        gw, _ = win.grads_unpacked()
        for m, g in enumerate(full["grad_w"]):
            if g is not None:
                assert nerr(gw[m], g) < 1e-3


@pytest.mark.parametrize("spec_fn,T,N", [(lambda: wl.lstm_net(40, [512], 61), 40, 17), (lambda: wl.elman_net(40, 1024, 61), 600, 3),
                                         (lambda: wl.elman_net(3, 1, 2), 60000, 9)])
def test_static_workspace_does_not_count_the_copies_of_ragged_tiles(spec_fn, T, N):
    """Windows that fit RNN_STATIC_WORKSPACE_BYTES but for the second copies of their exchanged tensors."""
    spec = spec_fn()
    w = wl.make_workload("static_ragged", spec, T=T, N=N, seed=75, scale=0.05)
    win, ref, got = outputs_both_ways(w)
    assert win.g.workspace_bytes(T, N) > 32 << 20
    for k in spec.output_nodes():
        assert np.array_equal(got[k], ref[k])


def test_static_call_of_an_element_wise_recurrence_needs_no_code_that_is_loaded_first():
    """Beyond eight streams such a recurrence can go frame by frame: the first call on a handle may be a static one; with the
    kernel loaded it is used.  Up to eight streams there is no such way, and the call is refused."""
    import torch
    from paper_1503_02852_amd import RnnError
    from paper_1503_02852_amd.runner import window_for
    spec = wl.lstm_net(11, [29], 5, output_recurrence=False)
    (out,) = spec.output_nodes()
    for N in (8, 12):
        w = wl.make_workload("static_first", spec, T=7, N=N, seed=83, scale=0.4, bias_scale=0.3)
        win = window_for(w)
        got = torch.full((w.T, N, spec.nodes[out]["dim"]), float("nan"), dtype=torch.float32, device=win.dev)
        call = lambda: win.g.forward_static(win.weights.data_ptr(), win._input_ptrs(), [got.data_ptr()], w.T, w.N, win._stream())
        if N == 8:
            with pytest.raises(RnnError):
                call()
            continue
        y, _ = go.forward(spec.nodes, spec.edges, w.weights, w.biases, w.inputs, w.T, N)
        for build in ("per_frame", "wave"):
            call()
            win.check()
            rec = [k for k in range(len(spec.nodes)) if win.g.step_build(k)[0] != "none"]
            assert rec and all(win.g.step_build(k)[0] == build for k in rec)
            assert nerr(got.cpu().numpy(), y[out]) < OUT_TOL
            win.forward()


def test_static_call_under_capture_with_copies_beyond_the_workspace():
    """A captured rnn_forward_static in the larger array, replayed with other work in between."""
    import torch
    spec = wl.lstm_net(8, [512], 4)
    w = wl.make_workload("static_capture", spec, T=40, N=17, seed=76, scale=0.05)
    win, ref, _ = outputs_both_ways(w)
    (o,) = spec.output_nodes()
    out = torch.zeros((w.T, w.N, 4), dtype=torch.float32, device=win.dev)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        win.g.forward_static(win.weights.data_ptr(), win._input_ptrs(), [out.data_ptr()], w.T, w.N, win._stream())
    for _ in range(3):
        out.fill_(float("nan"))
        win.forward()                  # eager, on the caller's workspace
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), ref[o])


def test_static_workspace_limits_and_preconditions():
    import torch
    from paper_1503_02852_amd.binding import RnnError
    from paper_1503_02852_amd.runner import window_for
    spec = wl.lstm_net(10, [48], 6)
    w = wl.make_workload("static_pre", spec, T=12, N=2, seed=73)
    win = window_for(w)
    (o,) = spec.output_nodes()
    out = torch.zeros((w.T, w.N, 6), dtype=torch.float32, device=win.dev)
    # a window beyond the static array's size is refused with a clear message
    with pytest.raises(RnnError) as ei:
        win.g.forward_static(win.weights.data_ptr(), win._input_ptrs(), [out.data_ptr()], 1 << 20, 2, win._stream())
    assert ei.value.code == -3 and "static workspace" in str(ei.value)
    # the kernels must have been loaded by an ordinary call before
    spec2 = wl.lstm_net(10, [44], 6)          # a width no other test uses: its step kernel is not in the process's cache
    w2 = wl.make_workload("static_cold", spec2, T=12, N=2, seed=74)
    cold = window_for(w2)
    with pytest.raises(RnnError) as ei:
        cold.g.forward_static(cold.weights.data_ptr(), cold._input_ptrs(), [out.data_ptr()], w2.T, w2.N, cold._stream())
    assert ei.value.code == -4 and "not been loaded" in str(ei.value)
    cold.forward()
    cold.g.forward_static(cold.weights.data_ptr(), cold._input_ptrs(), [out.data_ptr()], w2.T, w2.N, cold._stream())
    cold.check()
    # kernel-class timing would create events
    win.forward()
    ref = win.node_output(o).astype(np.float64)
    win.g.profile_enable(1)
    with pytest.raises(RnnError) as ei:
        win.g.forward_static(win.weights.data_ptr(), win._input_ptrs(), [out.data_ptr()], w.T, w.N, win._stream())
    assert ei.value.code == -4
    win.g.profile_enable(0)
    win.g.forward_static(win.weights.data_ptr(), win._input_ptrs(), [out.data_ptr()], w.T, w.N, win._stream())
    win.check()
    assert nerr(out.cpu().numpy(), ref) < OUT_TOL
