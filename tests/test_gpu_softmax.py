"""Row softmax and the cross-entropy output delta at the edges of the row widths that their kernels take."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("O", [1, 2, 63, 64, 65, 256, 257, 1023, 1024, 1025, 1027, 2047, 2048, 2049, 4096, 4097, 8191, 8192, 8193, 20480, 20483, 40960, 40963])
def test_softmax_and_delta_at_row_width_edges(O):
    from paper_1503_02852_amd.runner import window_for
    K, T, N = 3, 5, 3
    g = wl.GraphSpec()
    x = g.add_node(wl.INPUT, wl.LINEAR, K, name="x")
    o = g.add_node(wl.ADD, wl.SOFTMAX, O, is_output=wl.CROSS_ENTROPY, name="o")
    g.add_edge(x, o, wl.FULL, 0)
    w = wl.make_workload("softmax", g, T=T, N=N, seed=O, scale=2.0)
    tg = w.targets[o]
    tg.reshape(-1)[:4] = 0, O - 1, -1, min(O - 1, 4095)
    win = window_for(w)
    win.forward()
    win.bptt()
    loss = win.compute_grads(want_loss=True)
    win.check()
    X, W = w.inputs[0].reshape(T * N, K).astype(np.float64), w.weights[0].astype(np.float64)
    s, mag = X @ W.T, (np.abs(X) @ np.abs(W).T).max()
    d = s - s.max(axis=1, keepdims=True)
    ref = np.exp(d) / np.exp(d).sum(axis=1, keepdims=True)
    y = win.node_output(1).reshape(T * N, O)
    # relative: the product's roundings reach the exponent (K + 6 of mag, own and in the sum), the
    # exponential multiplies its argument by log2 e (three roundings of |d|), additions of one lane and across
    # lanes (at most 64 for these widths), a reciprocal and products
    rel = 2.0 ** -24 * (2 * (K + 6) * mag + 6 * np.abs(d) + 6 * np.abs(d).max() + 80)
    assert (np.abs(y - ref) <= rel * ref + 1e-37).all(), (np.abs(y - ref) / (rel * ref + 1e-37)).max()
    tg = tg.reshape(-1)
    hot = np.zeros((T * N, O), np.float32)
    hot[tg >= 0, tg[tg >= 0]] = 1.0
    want = np.where(tg[:, None] >= 0, y - hot, np.float32(0.0))
    assert (win.node_state_grad(1).reshape(T * N, O) == want).all()
    l = -np.log(y[tg >= 0, tg[tg >= 0]].astype(np.float64))
    # the logarithm: |result| times a few roundings, and 2^-21 near 1; a sum of up to four in fp32
    assert abs(loss - l.sum()) <= 2.0 ** -22 * (4 * np.abs(l).sum() + 2 * len(l))


@pytest.mark.parametrize("O,T", [(1025, 260), (1027, 601), (2048, 512), (2049, 512), (4097, 1100), (4100, 1024)])
def test_output_delta_of_many_rows_around_the_change_of_kernels(O, T):
    """Rows above 1,024 columns are taken whole by a wavefront each, or in segments by workgroups,
    depending on how many rows and columns there are."""
    from paper_1503_02852_amd.runner import window_for
    g = wl.GraphSpec()
    x = g.add_node(wl.INPUT, wl.LINEAR, 2, name="x")
    o = g.add_node(wl.ADD, wl.SOFTMAX, O, is_output=wl.CROSS_ENTROPY, name="o")
    g.add_edge(x, o, wl.FULL, 0)
    w = wl.make_workload("delta", g, T=T, N=1, seed=O)
    tg = w.targets[o].reshape(-1)
    tg[:4] = 0, O - 1, -1, 1024
    win = window_for(w)
    win.forward()
    win.bptt()
    loss = win.compute_grads(want_loss=True)
    y = win.node_output(1).reshape(T, O)
    hot = np.zeros((T, O), np.float32)
    hot[tg >= 0, tg[tg >= 0]] = 1.0
    assert (win.node_state_grad(1).reshape(T, O) == np.where(tg[:, None] >= 0, y - hot, np.float32(0.0))).all()
    l = -np.log(y[tg >= 0, tg[tg >= 0]].astype(np.float64))
    # a few roundings of each logarithm; sums of up to four in fp32, the rest in double
    assert abs(loss - l.sum()) <= 2.0 ** -22 * (4 * np.abs(l).sum() + 2 * len(l))


@pytest.mark.parametrize("T,N", [(1, 1), (9, 1), (65, 1), (130, 5), (700, 3), (300, 20)])
def test_sums_over_frames(T, N):
    """Bias and peephole gradients (sums over all frames of one and of two factors, one of them a frame back) and the
    loss, at row counts around the groups that a thread takes at once, against float64 on the GPU's own factors."""
    from paper_1503_02852_amd.runner import window_for
    spec = wl.lstm_net(4, [70], 9)
    w = wl.make_workload("sums", spec, T=T, N=N, seed=T + N, scale=0.4, bias_scale=0.3, masked_fraction=0.2)
    win = window_for(w)
    win.forward()
    win.bptt()
    loss = win.compute_grads(want_loss=True)
    gw, gb = win.grads_unpacked()

    def check(got, a, b):
        # a product and a sum over T N frames, each rounded by 2^-24 of the magnitudes' sum
        want, size = (a * b).sum(axis=(0, 1)), np.abs(a * b).sum(axis=(0, 1))
        assert (np.abs(got - want) <= (T * N + 4) * 2.0 ** -24 * size + 1e-37).all()

    sums = 0
    for k, node in enumerate(spec.nodes):
        if node["has_bias"]:
            check(gb[k], win.node_state_grad(k).astype(np.float64), 1.0)
            sums += 1
    for m, e in enumerate(spec.edges):
        if e["wkind"] == wl.DIAG and spec.nodes[e["dst"]]["kind"] == wl.ADD:
            y = np.zeros((T, N, 70))
            y[e["delay"]:] = win.node_output(e["src"])[:T - e["delay"]]
            check(gw[m], win.node_state_grad(e["dst"]).astype(np.float64), y)
            sums += 1
    assert sums >= 8
    (o,) = spec.output_nodes()
    tg = w.targets[o].reshape(-1)
    p = win.node_output(o).astype(np.float64).reshape(T * N, -1)[np.arange(T * N), np.maximum(tg, 0)]
    want = -np.log(p[tg >= 0]).sum()
    # the hardware logarithm's error (2 ulp of log2 near 1: 2^-22 absolute) per frame
    assert abs(loss - want) <= 2.0 ** -21 * max(1.0, T * N) + 1e-6 * want


@pytest.mark.parametrize("T,O", [(1, 3), (37, 130), (513, 256), (1023, 4096), (1100, 4096)])
def test_squared_error_sums_in_double(T, O):
    """The loss of up to several million elements against a double sum of the terms, each rounded to fp32 like the kernel's."""
    from paper_1503_02852_amd.runner import window_for
    spec = wl.GraphSpec()
    x = spec.add_node(wl.INPUT, wl.LINEAR, 4, name="x")
    o = spec.add_node(wl.ADD, wl.LINEAR, O, has_bias=True, is_output=wl.SQUARED_ERROR, name="y")
    spec.add_edge(x, o, wl.FULL, 0)
    w = wl.make_workload("squared", spec, T=T, N=1, seed=T, scale=0.4, bias_scale=0.3)
    win = window_for(w)
    win.forward()
    win.bptt()
    loss = win.compute_grads(want_loss=True)
    err = win.node_output(o) - w.targets[o].astype(np.float32)
    terms = (np.float32(0.5) * err * err).astype(np.float64)
    # every addition of the longest chain (a thread's terms, a wavefront, a workgroup, up to 2,048 workgroups) rounds by 2^-53
    assert abs(loss - terms.sum()) <= 2.0 ** -53 * (T * O / (512 * 256) + 2048 + 16 + 64) * terms.sum()


@pytest.mark.parametrize("T", [66576, 66577])
def test_output_delta_of_many_short_rows(T):
    """61 classes, as many rows as 512 workgroups take and one more: every row's delta and the loss."""
    from paper_1503_02852_amd.runner import window_for
    spec = wl.GraphSpec()
    x = spec.add_node(wl.INPUT, wl.LINEAR, 4, name="x")
    o = spec.add_node(wl.ADD, wl.SOFTMAX, 61, has_bias=True, is_output=True, name="y")
    spec.add_edge(x, o, wl.FULL, 0)
    w = wl.make_workload("rows", spec, T=T, N=1, seed=T, scale=0.4, bias_scale=0.3)
    w.targets[o][::7] = -1
    win = window_for(w)
    win.forward()
    win.bptt()
    loss = win.compute_grads(want_loss=True)
    y, tg = win.node_output(o).reshape(T, 61), w.targets[o].reshape(-1)
    used = tg >= 0
    want = np.where(used[:, None], y, np.float32(0.0))
    want[used, tg[used]] -= np.float32(1.0)
    assert np.array_equal(win.node_state_grad(o).reshape(T, 61), want)
    # the hardware logarithm's error (2 ulp of log2 near 1: 2^-22 absolute) per frame
    sum_ = -np.log(y[used, tg[used]].astype(np.float64)).sum()
    assert abs(loss - sum_) <= 2.0 ** -21 * T + 1e-6 * sum_
