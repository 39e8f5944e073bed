"""GPU parity of the matrix-core step kernels where neither the streams nor the units fill whole
16 x 16 tiles: the tile-blocked exchange tensors are padded, and stream groups may be unequal."""
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


@pytest.mark.parametrize("layers,N", [([29, 21], 21), ([18], 9)])
def test_ragged_windows_in_pieces_and_moved_ahead(monkeypatch, layers, N):
    """History frames of the padded exchange tensors, in both window forms."""
    monkeypatch.setitem(tw.WINDOW_NETS, "ragged", lambda: (wl.lstm_net(8, layers, 4), N))
    tw.test_window_computed_in_pieces_equals_the_window_at_once("ragged")
    tw.test_window_moved_ahead_with_carried_state("ragged")
