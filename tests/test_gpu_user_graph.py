"""Steps captured by the caller into a graph of its own: two steps (the buffers swap back), replayed
between eager calls.  A setter between two replays leaves nothing behind that the captured steps
would take for their own counts.  Every replay is checked against eager steps: cell types and bubble
ids exactly, gas volumes and masses to the rounding of the FP64 atomic sums.
"""
import numpy as np
import pytest

import paper_1712_07028_amd as fsl
from paper_1712_07028_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    fsl.load_library()


def agree(a, b):
    for k in (fsl.FIELD_FLAGS, fsl.FIELD_BUBBLE_ID):
        np.testing.assert_array_equal(a.get(k), b.get(k))
    ba, bb = a.bubbles(), b.bubbles()
    assert [x["alive"] for x in ba] == [x["alive"] for x in bb]
    for x, y in zip(ba, bb):
        for k in ("V", "M", "rho_g"):
            assert abs(x[k] - y[k]) <= 1e-10 * max(1.0, abs(y[k])), k


def test_replays_after_a_bubble_table_was_set():
    import torch

    w = W.bubble_column_small()
    g, e = fsl.Sim(w), fsl.Sim(w)
    g.step(4)
    e.step(4)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=g.stream):
        g.step(2)
    for _ in range(2):
        for _ in range(3):
            with torch.cuda.stream(g.stream):
                graph.replay()
            for _ in range(2):
                e.step(1)
            agree(g, e)
        b = e.bubbles()
        for s in (g, e):
            s.bubbles_set([x["M"] for x in b], list(range(len(b))), [x["alive"] for x in b])
    g.close()
    e.close()
