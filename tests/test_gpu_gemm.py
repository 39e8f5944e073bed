"""The batched products (forward, backward, weight gradients) at tile and chunk edges, each against
float64 on the operands that the GPU used, and with operands at the ends of the fp32 range."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


def linear_pair(K, H, O, delay):
    """x -> a -> o, both layers linear, squared error: nothing but products."""
    g = wl.GraphSpec()
    x = g.add_node(wl.INPUT, wl.LINEAR, K, name="x")
    a = g.add_node(wl.ADD, wl.LINEAR, H, name="a")
    o = g.add_node(wl.ADD, wl.LINEAR, O, is_output=wl.SQUARED_ERROR, name="o")
    g.add_edge(x, a, wl.FULL, delay)
    g.add_edge(a, o, wl.FULL, 0)
    return g


def check_product(got, A, B, what):
    """got = A B in fp32: n products and additions, each rounded by at most 2^-24 of the sum of
    magnitudes, and six more roundings for parts summed on their own and across workgroups."""
    A, B = A.astype(np.float64), B.astype(np.float64)
    bound = (A.shape[1] + 6) * 2.0 ** -24 * (np.abs(A) @ np.abs(B)) + 1e-37
    worst = (np.abs(got - A @ B) / bound).max()
    assert worst <= 1.0, (what, worst)


@pytest.mark.parametrize("K,H,O,T,N,delay", [(1, 1, 1, 1, 1, 0), (31, 33, 5, 7, 9, 0), (32, 127, 61, 129, 1, 0), (33, 129, 128, 16, 8, 1),
                                             (39, 250, 61, 50, 3, 2), (64, 130, 257, 65, 2, 0), (1050, 40, 30, 33, 1, 1), (4100, 96, 40, 40, 2, 0)])
def test_products_at_tile_and_chunk_edges(K, H, O, T, N, delay):
    from paper_1503_02852_amd.runner import window_for
    w = wl.make_workload("pair", linear_pair(K, H, O, delay), T=T, N=N, seed=K + H, scale=0.5)
    win = window_for(w)
    win.step()
    win.check()
    a, do, da = (v.reshape(T * N, -1) for v in (win.node_output(1), win.node_state_grad(2), win.node_state_grad(1)))
    x = np.concatenate([np.zeros((delay, N, K), np.float32), w.inputs[0]])[:T].reshape(T * N, K)
    gw, _ = win.grads_unpacked()
    check_product(a, x, w.weights[0].T, "x W'")
    check_product(win.node_output(2).reshape(T * N, -1), a, w.weights[1].T, "a W'")
    check_product(da, do, w.weights[1], "d W")
    check_product(gw[1], do.T, a, "d' a")
    check_product(gw[0], da.T, x, "d' x")


def test_infinities_nan_and_the_ends_of_the_range():
    """An infinity, a NaN or a value next to the largest reaches the results that fp32 arithmetic
    gives it, and no others; operands down to 2^-130 keep all their bits."""
    from paper_1503_02852_amd.runner import window_for
    K, H, T = 70, 140, 300
    w = wl.make_workload("pair", linear_pair(K, H, 9, 0), T=T, N=1, seed=3, scale=0.5)
    x = w.inputs[0].reshape(T, K)
    x[3, 5], x[130, 40], x[131, 69], x[200, 0] = np.inf, -np.inf, np.nan, np.finfo(np.float32).max
    x[201, 1] = -3.4e38
    for i, e in enumerate((-90, -100, -110, -118, -120, -124, -126, -130)):
        x[250 + i] *= np.float32(2.0 ** e)
    win = window_for(w)
    win.forward()
    a = win.node_output(1).reshape(T, H)
    with np.errstate(all="ignore"):
        exact = x.astype(np.float64) @ w.weights[0].T.astype(np.float64)
        ref = exact.astype(np.float32)
        size = np.abs(x).astype(np.float64) @ np.abs(w.weights[0].T).astype(np.float64)
    assert np.array_equal(np.isnan(a), np.isnan(ref)) and np.isnan(ref).any()
    inf = np.isinf(ref)
    assert inf.any() and np.array_equal(a[inf], ref[inf]) and not np.isinf(a[~inf & ~np.isnan(ref)]).any()
    # K products and K additions: 2^-24 of the sum of magnitudes each, or half of the subnormal spacing 2^-149
    ok = np.isfinite(ref)
    assert (np.abs(a[ok].astype(np.float64) - exact[ok]) <= (K + 6) * 2.0 ** -24 * size[ok] + K * 2.0 ** -149).all()


@pytest.mark.parametrize("K,H,O,T,N,delay", [(40, 256, 61, 96, 8, 1),          # one kind of tile per direction: of 64, 32 and 32
                                             (130, 1030, 260, 700, 5, 1),      # tiles of 128 with a remainder, gradients in parts
                                             (250, 250, 250, 1000, 3, 2),
                                             (520, 2050, 24, 1030, 2, 0),      # narrow gradients beside a wide one: two launches
                                             (5000, 520, 16, 200, 3, 0)])      # a long contraction added up over workgroups
def test_products_in_every_kind_of_tile(K, H, O, T, N, delay):
    test_products_at_tile_and_chunk_edges(K, H, O, T, N, delay)


@pytest.mark.parametrize("K,H,O,T,delay", [(2 ** 22 + 5, 3, 2, 3, 1), (2, 2 ** 22 + 3, 2, 2, 0)])
def test_rows_beyond_a_32_bit_tile(K, H, O, T, delay):
    test_products_at_tile_and_chunk_edges(K, H, O, T, 1, delay)


def test_more_products_than_one_launch_takes():
    """45 sources of one node (a launch takes 40 products) and 91 weight matrices (24)."""
    from oracle import graph_oracle as go
    from paper_1503_02852_amd.runner import window_for
    g = wl.GraphSpec()
    x = g.add_node(wl.INPUT, wl.LINEAR, 7, name="x")
    hs = [g.add_node(wl.ADD, wl.TANH, 3 + i % 40, name=f"h{i}") for i in range(45)]
    a = g.add_node(wl.ADD, wl.LINEAR, 33, name="a")
    o = g.add_node(wl.ADD, wl.LINEAR, 5, is_output=wl.SQUARED_ERROR, name="o")
    for i, h in enumerate(hs):
        g.add_edge(x, h, wl.FULL, 0)
        g.add_edge(h, a, wl.FULL, i % 3)
    g.add_edge(a, o, wl.FULL, 0)
    w = wl.make_workload("many", g, T=20, N=3, seed=9, scale=0.3)
    win = window_for(w)
    win.step()
    win.check()
    ref = go.forward_bptt(w.spec.nodes, w.spec.edges, w.weights, w.biases, w.inputs, w.targets, w.T, w.N)
    gw, _ = win.grads_unpacked()
    # at most 45 x 42 terms per sum, three products in a row: 2^-24 times the root of the terms, times 100 for cancellation
    for got, want in [(win.node_output(a), ref["y"][a]), (win.node_output(o), ref["y"][o])] + list(zip(gw, ref["grad_w"])):
        assert np.abs(got - want).max() <= 3e-4 * np.abs(want).max()


@pytest.mark.parametrize("act", [wl.LINEAR, wl.SIGMOID, wl.TANH, wl.RELU])
@pytest.mark.parametrize("K,H,O,T,N", [(5, 7, 3, 6, 1), (70, 130, 65, 130, 1), (90, 520, 300, 1100, 3), (4500, 40, 30, 9, 2)])
def test_nodes_finished_where_their_products_are_stored(K, H, O, T, N, act):
    """y = f(W x + b) of nodes that only products lead into, in every kind of tile, and where the products are split
    (the last case) by a program of its own; a second source, delayed, feeds the output node."""
    from oracle import graph_oracle as go
    from paper_1503_02852_amd.runner import window_for
    g = wl.GraphSpec()
    x = g.add_node(wl.INPUT, wl.LINEAR, K, name="x")
    a = g.add_node(wl.ADD, act, H, has_bias=True, name="a")
    o = g.add_node(wl.ADD, wl.SOFTMAX, O, has_bias=True, is_output=1, name="o")
    g.add_edge(x, a, wl.FULL, 0)
    g.add_edge(a, o, wl.FULL, 0)
    g.add_edge(a, o, wl.FULL, 1)
    w = wl.make_workload("finish", g, T=T, N=N, seed=K + O, scale=0.6 / np.sqrt(K), bias_scale=0.5)
    win = window_for(w)
    win.step()
    win.check()
    ref = go.forward_bptt(w.spec.nodes, w.spec.edges, w.weights, w.biases, w.inputs, w.targets, w.T, w.N)
    # sums of K and 2 H products, rounded by 2^-24 of their size each, through functions of slope 1 and below
    for k in (a, o):
        assert np.abs(win.node_output(k) - ref["y"][k]).max() <= (K + 2 * H + 20) * 2.0 ** -24 * max(1.0, np.abs(ref["y"][k]).max())
