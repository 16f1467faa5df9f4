"""Launches on the two sides of a rule's edge, or of one work split and the
next, must not differ in time by more than their work does.  Times are the
smallest of several replays of captured calls; each limit lies between what
both sides measured with and without the fault that the test names."""
import numpy as np
import pytest
import torch

from paper_2010_03166_amd import gnnprop as G
from paper_2010_03166_amd import runtime, synth

pytestmark = pytest.mark.gpu


def best_us(call, reps=8, rounds=7):
    """Time of one of `reps` captured calls, the best of `rounds` replays."""
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        for _ in range(reps):
            call()
    graph.replay()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = float("inf")
    for _ in range(rounds):
        a.record()
        graph.replay()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / reps * 1e3)
    return best


def gemm_us(ta, tb, M, N, K, flags=0, **kw):
    pad = lambda w: -(-w // 4) * 4
    A = torch.randn((K, pad(M)) if ta else (M, pad(K)), device="cuda")
    B = torch.randn((N, pad(K)) if tb else (K, pad(N)), device="cuda")
    C = torch.empty((M, pad(N)), device="cuda")
    ws = torch.empty(max(G.gnn_gemm_workspace_bytes(M, N, K), 256), dtype=torch.uint8,
                     device="cuda")
    return best_us(lambda: G.gnn_gemm(ta, tb, M, N, K, A, A.stride(0), B, B.stride(0), C,
                                      C.stride(0), flags, ws), **kw)


def test_long_rows_keep_float4_loads():
    """fp32 matrix cores, op(A) = A^T of 2^23 columns and of a few more: 10 %
    slower where the 32-bit offsets of another kernel decided (7 to 15 % over
    the kernels that index in 64 bits)."""
    below, above = (gemm_us(1, 0, (1 << 23) + d, 64, 64, G.GNN_FLAG_F32_MFMA, reps=2)
                    for d in (-8, 8))
    assert above < 1.05 * below, (below, above)


def test_second_k_segment_keeps_the_pipeline():
    """Input gradient of a layer of h = 208 (a first K segment that ends inside
    a stage of 32) against h = 224: 22 % dearer when all of the second segment
    took the guarded loop."""
    n, f = 8000, 256
    dg = runtime.DeviceGraph(synth.identity_graph(n))
    dg.prepare()
    us = {}
    for h in (208, 224):
        w = np.full((f, h), 0.01, np.float32)
        st = runtime.SageStack(dg, [synth.LayerParams(w, w)], f)
        x, dy = torch.randn((n, f), device="cuda"), torch.randn((n, 2 * h), device="cuda")
        us[h] = float("inf")
        for _ in range(5):
            st.forward(x)
            G.gnn_timer_enable(True)
            G.gnn_timer_reset()
            for _ in range(20):
                st.backward(dy)
            torch.cuda.synchronize()
            ms, launches, _ = G.gnn_timer_read("gemm_nt")
            G.gnn_timer_enable(False)
            us[h] = min(us[h], ms / launches * 1e3)
    assert us[208] < 1.15 * us[224], us


@pytest.mark.parametrize("shape,other,limit", [
    # one K range after the other on few CUs, or 16 parts of one stage and
    # their reduction: 1.37 times the time of a K more than twice as deep, now 0.9
    ((512, 41, 256), (512, 41, 602), 1.1),
    # 32 and 42 parts of one or two stages: 2.4 times the shallow product's
    # time, now 1.4
    ((1000, 256, 602), (1000, 256, 64), 1.9),
    ((700, 200, 1024), (700, 200, 41), 1.9),
])
def test_few_tiles_over_a_long_k(shape, other, limit):
    a, b = gemm_us(0, 0, *shape), gemm_us(0, 0, *other)
    assert a < limit * b, (a, b)


def _capped_graph(n, deg, kmax, seed=1):
    edges = synth.chung_lu_edges(n, 2.1, deg, kmax, np.random.default_rng(seed))
    g = runtime.DeviceGraph(synth.symmetric_csr(n, edges))
    g.prepare()
    return g


def spmm_us(g, w, ld):
    x, y = torch.randn(g.n * ld, device="cuda"), torch.empty(g.n * ld, device="cuda")
    csr = g.struct()
    return best_us(lambda: G.gnn_spmm(csr, 0, w, x, ld, y, ld, None))


def test_slices_leave_no_xcd_idle():
    """160 columns are five slices: 0.85 of the time of 256 columns when three
    of eight XCDs had empty ones, now 0.58."""
    g = _capped_graph(50000, 40.0, 1000)
    a, b = spmm_us(g, 160, 160), spmm_us(g, 256, 256)
    assert a < 0.72 * b, (a, b)


def test_narrow_slices_not_on_small_graphs():
    """24 columns of a 1,000-node graph: 1.4 times the time of 144 columns in
    slices of 16 columns, as long in one slice."""
    g = _capped_graph(1000, 10.0, 999)
    a, b = spmm_us(g, 24, 32), spmm_us(g, 144, 144)
    assert a < 1.2 * b, (a, b)


def test_wide_unaligned_rows_stay_one_pass():
    """514 columns in rows off 16-byte alignment: 1.8 times the time of 450
    when a lane group of 64 had to walk each slice twice, now 0.7."""
    g = _capped_graph(1000, 10.0, 999)
    a, b = spmm_us(g, 514, 514), spmm_us(g, 450, 450)
    assert a < 1.2 * b, (a, b)
