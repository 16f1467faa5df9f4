"""Split products whose B comes as ready pieces (M >= 512): every tile width,
whole and split tiles, partial stages and edges, against the double-precision
product.

Bound, per element: an output adds up 6 ceil(K / 32) piece products, each in at
most two steps that lose up to 2^-23 of a partial sum, which is at most
(|A| |B|)[i, j]; the pieces left out are below 2^-24 of each product, and a
reduction over parts adds a rounding per part (fewer than 8 + the steps)."""
import numpy as np
import pytest
import torch

from paper_2010_03166_amd import gnnprop as G
from paper_2010_03166_amd import runtime, synth

pytestmark = pytest.mark.gpu

SHAPES = [
    (512, 1, 1), (512, 16, 31), (513, 64, 32), (640, 63, 33),      # narrow, partial stages
    (600, 65, 40), (1000, 96, 96), (1023, 97, 127), (700, 129, 64),
    (1000, 256, 256),   # few tiles: whole, chained sums
    (2000, 200, 500),   # whole, 64 columns, chained
    (4000, 41, 1000),   # split along K, 64 columns
    (8000, 96, 41),     # two stages, the last one partial
    (8000, 602, 70),    # 96 columns
    (8003, 512, 200),   # two blocks per CU, moved-back rows
    (20000, 600, 65),   # more tiles than slots
]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("pad", [0, 1])
def test_split_planes(M, N, K, ta, tb, pad):
    gen = torch.Generator().manual_seed(M + 3 * N + 7 * K)
    a = torch.randn((M, K), generator=gen)
    b = torch.randn((K, N), generator=gen)

    def stored(x, trans):
        x = x.T if trans else x
        # padded to float4 rows, or off them
        ld = -(-x.shape[1] // 4) * 4 + pad
        buf = torch.full((x.shape[0], ld), float("nan"))
        buf[:, : x.shape[1]] = x
        return buf.cuda()

    A, B = stored(a, ta), stored(b, tb)
    ldc = -(-N // 4) * 4 + pad
    C = torch.full((M, ldc), float("nan"), device="cuda")
    ws = torch.empty(max(G.gnn_gemm_workspace_bytes(M, N, K), 256), dtype=torch.uint8,
                     device="cuda")
    G.gnn_gemm(ta, tb, M, N, K, A, A.stride(0), B, B.stride(0), C, ldc, 0, ws)
    torch.cuda.synchronize()
    got = C.cpu().numpy().astype(np.float64)
    assert np.isnan(got[:, N:]).all()  # nothing past the row's end
    ad, bd = a.numpy().astype(np.float64), b.numpy().astype(np.float64)
    err = np.abs(got[:, :N] - ad @ bd)
    bound = (12 * -(-K // 32) + 8) * 2.0 ** -23 * (np.abs(ad) @ np.abs(bd))
    assert (err <= bound).all(), float((err / bound).max())


@pytest.mark.parametrize("M,N,K,shared,unbroken", [
    (6600, 1536, 600, 3.16e-7, 3.65e-7), (20000, 512, 400, 2.55e-7, 2.94e-7),
    (20000, 1024, 602, 3.48e-7, 3.69e-7)])
def test_whole_tiles_for_shared_ones_keep_partial_sums(M, N, K, shared, unbroken):
    """More than 512 tiles of 128 x 128, where the general work split shares
    tiles over blocks.  Relative 2-norm errors measured: `shared` with its
    partial sums, `unbroken` with all of K in one chain of the matrix cores,
    which truncate what they shift out (below 1e-7 when the sums begin anew
    every 32 k).  The limit lies halfway between the two."""
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn((M, -(-K // 4) * 4), device="cuda", generator=gen)
    B = torch.randn((K, N), device="cuda", generator=gen)
    C = torch.empty((M, N), device="cuda")
    ws = torch.empty(max(G.gnn_gemm_workspace_bytes(M, N, K), 256), dtype=torch.uint8,
                     device="cuda")
    G.gnn_gemm(0, 0, M, N, K, A, A.stride(0), B, N, C, N, 0, ws)
    ref = A[:, :K].double() @ B.double()
    assert ((C.double() - ref).norm() / ref.norm()).item() < (shared + unbroken) / 2


@pytest.mark.parametrize("h", [16, 31, 32, 48, 80, 97, 208])
@pytest.mark.parametrize("n,f", [(640, 256), (1000, 601), (8003, 300)])
def test_two_segment_input_gradient(n, f, h):
    """dX = G_s W_self^T + T W_neigh^T in one launch, K segments of every
    depth within a stage of 32 (on the identity graph T = G_n).  Bound as
    above, over the stages of both segments."""
    dg = runtime.DeviceGraph(synth.identity_graph(n))
    dg.prepare()
    gen = torch.Generator().manual_seed(n + f + h)
    rows = lambda w: torch.full((n, -(-w // 16) * 16), float("nan"), device="cuda")[:, :w]
    X, Y, dY, dX = rows(f), rows(2 * h), rows(2 * h), rows(f)
    dY.copy_(torch.randn((n, 2 * h), generator=gen))
    X.copy_(torch.randn((n, f), generator=gen))
    Ws, Wn = (torch.randn((f, h), generator=gen).cuda() for _ in range(2))
    dWs, dWn = torch.empty_like(Ws), torch.empty_like(Wn)
    lay = G.make_layer(f, h, X.stride(0), Y.stride(0), dX.stride(0), 2, G.GNN_FLAG_DY_MASKED)
    csr = dg.struct()
    saved, ws = (torch.empty(max(b, 256), dtype=torch.uint8, device="cuda") for b in
                 (G.gnn_prop_saved_bytes(csr, lay), G.gnn_prop_workspace_bytes(csr, lay)))
    fwd = G.make_layer(f, h, X.stride(0), Y.stride(0), dX.stride(0), 2, 0)
    G.gnn_prop_fwd(csr, fwd, X, Ws, Wn, None, None, Y, saved, ws)
    G.gnn_prop_bwd(csr, lay, X, Ws, Wn, Y, dY, saved, dX, dWs, dWn, None, None, ws)
    torch.cuda.synchronize()
    g = dY.cpu().double()
    w = torch.cat([Ws, Wn], 1).cpu().double()
    err = (dX.cpu().double() - g @ w.T).abs()
    bound = (24 * -(-h // 32) + 8) * 2.0 ** -23 * (g.abs() @ w.abs().T)
    assert (err <= bound).all(), float((err / bound).max())


@pytest.mark.parametrize("f,h", [(16, 512), (1024, 16), (512, 16), (16, 96), (602, 512)])
@pytest.mark.parametrize("order", [1, 2])
def test_layer_with_pieces_in_one_direction_only(f, h, order):
    """Wide outputs of few stages go to the kernel that splits the weight
    itself, forward and input gradient each by its own shape (identity graph;
    bounds as above)."""
    n = 6001
    dg = runtime.DeviceGraph(synth.identity_graph(n))
    dg.prepare()
    gen = torch.Generator().manual_seed(f + h)
    st = runtime.SageStack(dg, [synth.LayerParams(
        *(torch.randn((f, h), generator=gen).numpy() for _ in range(2)))], f, order=order)
    L = st.layers[0]
    x = runtime.padded(torch.randn((n, f), generator=gen).cuda(), -(-f // 16) * 16)
    y = st.forward(x)
    dy = runtime.padded(torch.randn((n, 2 * h), generator=gen).cuda(), L["Y"].stride(0))
    dx = st.backward(dy)
    torch.cuda.synchronize()
    w = torch.cat([L["W_self"], L["W_neigh"]], 1).cpu().double()
    xd, g = x.cpu().double(), dy.cpu().double() * (y.cpu() > 0)

    def check(got, a, b, k):
        err = (got.cpu().double() - (a @ b).clamp_min(0) if got is y else
               got.cpu().double() - a @ b).abs()
        bound = (12 * -(-k // 32) + 16) * 2.0 ** -23 * (a.abs() @ b.abs())
        assert (err <= bound).all(), float((err / bound.clamp_min(1e-30)).max())

    check(y, xd, w, f)
    check(dx, g, w.T, 2 * h + 64)
    check(L["dW_self"], xd.T, g[:, :h], n)
    check(L["dW_neigh"], xd.T, g[:, h:], n)


# every way the work split takes a product of 512 rows and more
WAYS = [
    (512, 64, 64),      # whole tiles of 64 columns, one chain over K
    (50000, 96, 41),    # of 96
    (8000, 1024, 602),  # of 128
    (1000, 602, 128),   # 64 columns in place of parts: every stage from zero
    (2000, 1200, 200),  # in place of stream-K
    (1000, 256, 602),   # K over several blocks, every stage from zero
    (6000, 301, 1500),  # the same in place of stream-K
    (512, 64, 602),     # K over several blocks, 64 columns
    (8000, 129, 1024),  # 96
    (5000, 301, 4096),  # 128
    (512, 41, 256),     # the kernel that splits both operands itself: parts
    (8000, 512, 200),   # whole tiles
    (50000, 512, 1024),  # stream-K
]


def _padded(x, ta):
    x = x.T if ta else x
    buf = torch.full((x.shape[0], -(-x.shape[1] // 4) * 4), float("nan"), device="cuda")
    buf[:, : x.shape[1]] = x
    return buf


def _product(a, b, ta, tb):
    M, K = a.shape
    N = b.shape[1]
    A, B = _padded(a, ta), _padded(b, tb)
    C = torch.full((M, N), float("nan"), device="cuda")
    ws = torch.empty(max(G.gnn_gemm_workspace_bytes(M, N, K), 256), dtype=torch.uint8,
                     device="cuda")
    G.gnn_gemm(ta, tb, M, N, K, A, A.stride(0), B, B.stride(0), C, N, 0, ws)
    return C


@pytest.mark.parametrize("M,N,K", WAYS)
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
def test_every_way_of_splitting_the_work(M, N, K, ta, tb):
    gen = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K)
    a = torch.randn((M, K), device="cuda", generator=gen)
    b = torch.randn((K, N), device="cuda", generator=gen)
    err = (_product(a, b, ta, tb).double() - a.double() @ b.double()).abs()
    bound = (12 * -(-K // 32) + 8) * 2.0 ** -23 * (a.double().abs() @ b.double().abs())
    assert (err <= bound).all(), float((err / bound).max())


@pytest.mark.parametrize("M,N,K", WAYS)
@pytest.mark.parametrize("ta", [0, 1])
@pytest.mark.parametrize("dense", ["a", "b"])
def test_every_operand_bit_counts(M, N, K, ta, dense):
    """One operand holds numbers of 24 significand bits (1 + 2^-9 + 2^-18 +
    2^-23 times powers of two: three pieces, none 0), the other picks one of
    them per output with a power of two: each result is exact in fp32, and a
    product of pieces left out or doubled shows in every element."""
    rng = np.random.default_rng(M + N + K)
    sig = 1.0 + 2.0 ** -9 + 2.0 ** -18 + 2.0 ** -23
    full = lambda r, c: (sig * rng.choice([1.0, -1.0], size=(r, c))
                         * np.ldexp(1.0, rng.integers(-3, 4, size=(r, c)))).astype(np.float32)
    if dense == "a":
        a, b = full(M, K), np.zeros((K, N), np.float32)
        k, w = rng.integers(0, K, N), np.ldexp(1.0, -rng.integers(0, 3, N)).astype(np.float32)
        b[k, np.arange(N)] = w
        want = a[:, k] * w
    else:
        a, b = np.zeros((M, K), np.float32), full(K, N)
        k, w = rng.integers(0, K, M), np.ldexp(1.0, -rng.integers(0, 3, M)).astype(np.float32)
        a[np.arange(M), k] = w
        want = b[k] * w[:, None]
    got = _product(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), ta, 0)
    assert torch.equal(got, torch.from_numpy(want).cuda())
