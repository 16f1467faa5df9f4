"""Column slices of the aggregation: every number of slices and lane-group
width, ragged row ends, and buffers that end with the last row's last column,
against the oracle (and the 1e-5 that gnn_spmm is held to elsewhere)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2010_03166_amd import gnnprop as G
from paper_2010_03166_amd import runtime, synth

pytestmark = pytest.mark.gpu

TOL = 1e-5
SMALL = synth.power_law_graph(700, 2.1, 12.0, seed=11)
MIDDLE = synth.power_law_graph(9000, 2.1, 20.0, seed=12)  # 739 windows
LARGE = synth.workload_graph(synth.WORKLOADS["cl2.1-n20000-f200-h512-L5"])  # 2,422 windows


def _exact_rows(rows, cols, ld, fill=None):
    """rows x cols view of stride ld over a buffer that ends with the last
    element, NaN in the padding."""
    buf = torch.full(((rows - 1) * ld + cols,), float("nan"), device="cuda")
    view = buf.as_strided((rows, cols), (ld, 1))
    if fill is not None:
        view.copy_(torch.from_numpy(fill))
    return view


@pytest.mark.parametrize("graph,w", [
    ("small", w) for w in (15, 17, 33, 50, 64, 66, 127, 130, 199, 258, 301, 390, 513, 602, 700, 1030)
] + [("middle", w) for w in (50, 64, 101, 128, 161, 256, 321)]
  + [("large", w) for w in (50, 64, 101, 200, 256, 257, 300, 510, 602)])
@pytest.mark.parametrize("transpose", [0, 1])
def test_spmm_slices(graph, w, transpose):
    g = {"small": SMALL, "middle": MIDDLE, "large": LARGE}[graph]
    dg = runtime.DeviceGraph(g)
    dg.prepare()
    x = np.random.default_rng(w + transpose).standard_normal((g.n, w)).astype(np.float32)
    ld = -(-w // 4) * 4 + 4 * (w % 3)
    xin, out = _exact_rows(g.n, w, ld, x), _exact_rows(g.n, w, ld)
    G.gnn_spmm(dg.struct(), transpose, w, xin, ld, out, ld, None)
    torch.cuda.synchronize()
    ref = O.spmm_transpose(g, x) if transpose else O.spmm(g, x)
    got = out.cpu().numpy().astype(np.float64)
    assert np.abs(got - ref).max() <= TOL * np.abs(ref).max()
    if ld > w:  # the padding between rows stays untouched
        gap = out.as_strided((g.n - 1, ld - w), (ld, 1), w)
        assert torch.isnan(gap).all()


def test_two_windows_per_workgroup_many_slices():
    """More than 16,384 workgroups (2,422 windows x 8 slices)."""
    assert -(-LARGE.nnz // 256) * 8 > 16384
    test_spmm_slices("large", 604, 0)
    test_spmm_slices("large", 640, 1)


@pytest.mark.parametrize("w", [31, 33, 257, 511, 513, 639, 641, 1025, 2049, 2113])
@pytest.mark.parametrize("transpose", [0, 1])
def test_float_lanes(w, transpose):
    """Rows off 16-byte alignment: eight slices, slices of 32 and 64 columns
    (more of them than XCDs), and wider ones."""
    dg = runtime.DeviceGraph(SMALL)
    dg.prepare()
    x = np.random.default_rng(w + transpose).standard_normal((SMALL.n, w)).astype(np.float32)
    xin, out = _exact_rows(SMALL.n, w, w, x), _exact_rows(SMALL.n, w, w)
    G.gnn_spmm(dg.struct(), transpose, w, xin, w, out, w, None)
    torch.cuda.synchronize()
    ref = O.spmm_transpose(SMALL, x) if transpose else O.spmm(SMALL, x)
    got = out.cpu().numpy().astype(np.float64)
    assert np.abs(got - ref).max() <= TOL * np.abs(ref).max()
