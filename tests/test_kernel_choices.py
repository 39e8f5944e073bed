"""Which variant of a recurrent-step kernel a layer gets, read off the generated sources (the run-time compiler needs no GPU)."""
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import sys
import workloads as wl
from paper_1503_02852_amd import Graph
net, hidden, N = sys.argv[1].split(":")
hidden = [int(h) for h in hidden.split(",")]
spec = wl.elman_net(7, hidden[0], 5) if net == "elman" else wl.lstm_net(7, hidden, 5, output_recurrence=net != "element_wise")
Graph(spec.node_array(), spec.edge_array()).specialise(int(N))
"""


def sources(tmp_path, shapes, **env):
    """Per shape the sources of its forward and its backward launch (one of them, if they are the same); a process each, since a source is generated once."""
    clean = {k: v for k, v in os.environ.items() if not k.startswith("RNNG_")}
    got = []
    for i, shape in enumerate(shapes):
        d = tmp_path / str(i)
        d.mkdir()
        subprocess.run([sys.executable, "-c", CHILD, shape], check=True, cwd=ROOT, env={**clean, **env, "RNNG_JIT_DUMP": str(d)})
        got.append([(d / f).read_text() for f in sorted(os.listdir(d), key=lambda f: int(re.findall(r"_(\d+)\.hip", f)[0]))])
        assert 1 <= len(got[-1]) <= 2, shape
    return got


def constant(source, name):
    (value,) = set(re.findall(rf"\b{name} = (\w+)", source))
    return int(value.rstrip("ul"))


@pytest.mark.parametrize("local,ew", [("1", "1"), ("1", "0"), ("0", "1")])
def test_exchange_inside_one_xcd_and_wavefronts_for_the_element_wise_program(tmp_path, local, ew):
    shapes = ["lstm:18:33", "lstm:250:20"] if ew == "1" else ["lstm:3:9", "elman:41:140"]
    for shape, both in zip(shapes, sources(tmp_path, shapes, RNNG_MSTEP_LOCAL=local, RNNG_MSTEP_EW=ew)):
        for source in both:
            assert "mstep_kernel_body<grp0" in source, shape
            assert (constant(source, "LG") > 0) == (local == "1"), shape
            assert (constant(source, "NE") > 0) == (ew == "1"), shape
            assert (constant(source, "HOLD") > 0) == (local == "0"), shape


def test_resident_chunks_of_streamed_weights(tmp_path):
    """Of 17 chunks, the last one 4 columns wide, 7 in registers (that one among them) and 4 in LDS; of two chunks one each."""
    shapes = ["elman:2052:9", "elman:132:16"]
    expected = {"elman:2052:9": (7, 4), "elman:132:16": (1, 1)}
    for shape, both in zip(shapes, sources(tmp_path, shapes, RNNG_STEP_BUILD="stream", RNNG_SMSTEP_RESIDENT="1")):
        for source in both:
            assert "smstep_kernel_body" in source and (constant(source, "PR"), constant(source, "LRES")) == expected[shape], shape


def test_element_wise_recurrences_have_a_kernel_of_their_own(tmp_path):
    """A thread per stream and unit: forward at any number of streams, backward from nine on, below with many units (else on the lanes of the register build)."""
    shapes = {"element_wise:7:4": False, "element_wise:511:6": False, "element_wise:512:6": True, "element_wise:99:8": False, "element_wise:100:8": True, "element_wise:20:9": True}
    for (shape, expected), (forward, backward) in zip(shapes.items(), sources(tmp_path, list(shapes))):
        assert "estep_kernel_body" in forward, shape
        assert ("estep_kernel_body" in backward) == expected, shape


def test_four_streams_backward_exchange_inside_one_xcd_before_registers_of_two(tmp_path):
    """An LSTM layer whose weights take the registers of two XCDs: at four streams the matrix cores of one are ahead."""
    ((_, backward),) = sources(tmp_path, ["lstm:290:4"])
    assert "mstep_kernel_body<grp0" in backward and constant(backward, "LG") > 0


def test_streamed_weights_keep_residents_only_where_they_pay(tmp_path):
    """Forward / backward: 16 streams; the cache's size at 33; a walk left with one chunk in flight (20 streams); more weights than the cache and their residents hold (33)."""
    shapes = {"lstm:3200:16": (True, False), "lstm:4096:33": (True, True), "lstm:3584:20": (False, False), "elman:9216:33": (False, False)}
    for shape, both in zip(shapes, sources(tmp_path, list(shapes))):
        assert all("smstep_kernel_body" in source for source in both), shape
        assert tuple(constant(source, "PR") > 0 for source in (both[0], both[-1])) == shapes[shape], shape


def test_three_tiles_of_streams_keep_one_source_in_registers(tmp_path):
    """LSTM backward, four sources: a smaller unit chunk rather than two of them in registers, which spilled others."""
    ((_, backward),) = sources(tmp_path, ["lstm:1500:33"])
    assert "mstep_kernel_body<grp0" in backward and constant(backward, "MT") == 3
    assert bin(constant(backward, "REGMASK")).count("1") == 1
