"""Workloads on which this framework's speed is measured.

Each case is one piece of work that a training program hands to the library:
layers of every kind forward and backward, a two-layer stack on a small
subgraph, a whole training iteration, and the induction of a minibatch
subgraph.  `listed()` has the sizes of the paper's setting (8,000-node
subgraphs, hidden 512 per half, and the smaller and larger ones that the
benchmark also runs), `draw(rng)` gives more cases over the same ranges.

ReLU decisions.  An output that lies within rounding of 0 has no decided
ReLU derivative, and a single one decided otherwise outweighs every rounding
error of a gradient.  The upstream gradients drawn here are therefore 0 where
the pre-activation is that close to the kink; everything else about them is
N(0, 1).
"""
import numpy as np
import torch

from paper_2010_03166_amd import gnnprop as G
from paper_2010_03166_amd import runtime, synth

ALPHA = 0.2   # GAT's LeakyReLU slope
LR = 0.05     # SGD (Adam's first step is the sign of a gradient, rounding and all)


def listed():
    return [
        # the smallest call: a 1,000-node subgraph, two layers of 128 per
        # half, where launches and latency count
        dict(name="sage_stack_1k", kind="stack", graph="er", n=1000, deg=10.0, f=50, h=128,
             layers=2, mode="f32", bias=False),
        # first layer on a frontier-sampled 8,000-node subgraph with
        # Reddit-like 602-wide features (order A (X W), unaligned width)
        dict(name="sage_8k_f602", kind="sage", graph="cl", n=8000, deg=15.0, f=602, h=512,
             mode="f32", bias=False),
        # a hidden layer of the same stack: 2 x 512 in, 2 x 512 out
        dict(name="sage_8k_hidden", kind="sage", graph="cl", n=8000, deg=15.0, f=1024, h=512,
             mode="f32", bias=False),
        # odd and ragged sizes, biases, order (A X) W
        dict(name="sage_ragged", kind="sage", graph="cl", n=6001, deg=20.0, f=199, h=301,
             mode="f32", bias=True),
        # first layer of a deep network on a 20,000-node subgraph with
        # 200-wide features: aggregation-heavy, order (A X) W
        dict(name="sage_20k_f200", kind="sage", graph="cl", n=20000, deg=30.0, f=200, h=512,
             mode="f32", bias=False),
        # the largest: a hidden layer of 2 x 1,024 on a skewed 50,000-node
        # subgraph
        dict(name="sage_50k_hidden", kind="sage", graph="cl", n=50000, deg=40.0, f=2048, h=1024,
             mode="f32", bias=False),
        # a hidden layer with bf16 products
        dict(name="sage_8k_bf16", kind="sage", graph="cl", n=8000, deg=20.0, f=1024, h=512,
             mode="bf16", bias=False),
        # the other layer kinds on the 8,000-node subgraph
        dict(name="gcn_8k", kind="gcn", graph="cl", n=8000, deg=15.0, f=602, h=512,
             mode="f32", bias=True),
        dict(name="mixhop_8k", kind="mixhop", graph="cl", n=8000, deg=15.0, f=602, h=256, K=2,
             mode="f32", bias=False),
        dict(name="gat_8k", kind="gat", graph="cl", n=8000, deg=15.0, f=602, h=512,
             mode="f32", bias=False),
        # one whole training iteration on a new subgraph: its preparation,
        # two layers, classifier, loss, backward and the weight update
        dict(name="train_8k", kind="train", graph="cl", n=8000, deg=15.0, f=602, h=512,
             layers=2, C=41, mode="f32", bias=False),
        # a frontier-sampled node list to a minibatch subgraph with its
        # features and labels
        dict(name="induce_8k", kind="induce", scale=17, deg=16.0, m=1000, n=8000, f=50, C=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["sage", "sage", "sage", "sage", "gcn", "mixhop", "gat", "stack", "train",
                       "induce"])
    if kind == "induce":
        return dict(kind=kind, scale=rng.randint(14, 17), deg=16.0, m=_log_int(rng, 50, 1000),
                    n=_log_int(rng, 1000, 8000), f=rng.randint(20, 700), C=rng.randint(2, 121))
    c = dict(kind=kind, graph="cl", n=_log_int(rng, 700, 20000),
             deg=round(8.0 + 24.0 * rng.random(), 1), f=_log_int(rng, 48, 1100),
             h=_log_int(rng, 48, 520), mode=rng.choice(["f32", "f32", "f32", "bf16"]),
             bias=rng.random() < 0.3)
    if kind == "gat":  # no bias; bf16 scores leave the attention's own kinks undecided
        c["mode"] = "f32"
        c["bias"] = False
    if rng.random() < 0.5:  # widths that networks are usually given
        c["h"] = max(64, c["h"] // 64 * 64)
        c["f"] = max(32, c["f"] // 32 * 32)
    if kind == "mixhop":
        c["K"], c["h"] = rng.randint(1, 3), max(32, c["h"] // 2)
    if kind in ("stack", "train"):
        c.update(n=min(c["n"], 8000), layers=rng.randint(2, 3), mode="f32", bias=False)
    if kind == "train":
        c["C"] = rng.randint(7, 121)
    return c


# ---------------------------------------------------------------- inputs

def _flags(case):
    return G.GNN_FLAG_BF16 if case["mode"] == "bf16" else 0


def _graph(case, seed):
    n, deg = case["n"], case["deg"]
    values = "sym-normalized" if case["kind"] in ("gcn", "mixhop") else "row-normalized"
    rng = np.random.default_rng([seed, 1])
    if case["graph"] == "er":
        edges = synth.er_edges(n, deg, rng)
    else:
        gamma, kmax = (1.9, 5000) if n > 30000 else (2.1, 1000)
        edges = synth.chung_lu_edges(n, gamma, deg, min(kmax, n - 1), rng)
    return synth.symmetric_csr(n, edges, True, values)


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(n, f, gen):
    """n x f floats N(0, 1) at the row stride the runtime uses (16 floats)."""
    buf = torch.zeros((n, -(-f // 16) * 16), device="cuda")
    buf[:, :f] = torch.randn((n, f), device="cuda", generator=gen)
    return buf[:, :f]


def _glorot(f, h, gen):
    a = (6.0 / (f + h)) ** 0.5
    return (torch.rand((f, h), device="cuda", generator=gen) * 2 - 1) * a


def _inputs(case, seed):
    """The tensors of one layer (or stack) call, from the seed alone."""
    gen = _gen(seed)
    n, f, h, kind = case["n"], case["f"], case["h"], case["kind"]
    d = {"csr": _graph(case, seed), "X": _normal(n, f, gen), "W": [], "b": []}
    if kind in ("stack", "train", "sage"):
        fi = f
        for _ in range(case.get("layers", 1)):
            d["W"].append((_glorot(fi, h, gen), _glorot(fi, h, gen)))
            d["b"].append((0.1 * torch.randn(h, device="cuda", generator=gen),
                           0.1 * torch.randn(h, device="cuda", generator=gen))
                          if case["bias"] else (None, None))
            fi = 2 * h
        width = 2 * h
    else:
        width = (case["K"] + 1) * h if kind == "mixhop" else h
        d["W"] = _glorot(f, width, gen)
        d["b"] = 0.1 * torch.randn(width, device="cuda", generator=gen) if case["bias"] else None
        if kind == "gat":
            d["a"] = torch.randn(2 * h, device="cuda", generator=gen) * (0.5 / h) ** 0.5
    d["dY"] = _normal(n, width, gen)
    if kind == "train":
        C = case["C"]
        d["W_mlp"] = _glorot(width, C, gen)
        cls = torch.randint(C, (n,), device="cuda", generator=gen)
        d["T"] = torch.zeros((n, C), device="cuda")
        d["T"][torch.arange(n, device="cuda"), cls] = 1.0
    return d


class _Adj:
    """The subgraph's matrix in plain torch: products over its entries."""

    def __init__(self, csr, dtype):
        self.n = csr.n
        self.rows = torch.from_numpy(np.repeat(np.arange(csr.n), csr.degrees())).cuda()
        self.cols = torch.from_numpy(csr.indices.astype(np.int64)).cuda()
        self.vals = torch.from_numpy(csr.values).cuda().to(dtype)

    def mul(self, X, transpose=False, vals=None):
        r, c = (self.cols, self.rows) if transpose else (self.rows, self.cols)
        v = (self.vals if vals is None else vals)[:, None]
        out = torch.zeros((self.n, X.shape[1]), dtype=X.dtype, device=X.device)
        for k in range(0, X.shape[1], 128):
            part = torch.zeros((self.n, min(128, X.shape[1] - k)), dtype=X.dtype, device=X.device)
            part.index_add_(0, r, v * X[:, k: k + 128][c])
            out[:, k: k + 128] = part
        return out


def _layer_z(case, d, A, dt, X=None, i=0):
    """Pre-activations of a layer in precision dt (GAT: and its attention)."""
    X = d["X"].to(dt) if X is None else X
    kind, h = case["kind"], case["h"]
    if kind in ("sage", "stack", "train"):
        Ws, Wn = (w.to(dt) for w in d["W"][i])
        # A (X W) or (A X) W: equal; the narrower one is the cheaper
        nb = A.mul(X @ Wn) if X.shape[1] > h else A.mul(X) @ Wn
        z = torch.cat([X @ Ws, nb], 1)
        if d["b"][i][0] is not None:
            z = z + torch.cat(d["b"][i]).to(dt)
        return z
    W = d["W"].to(dt)
    if kind == "gat":
        P, a = X @ W, d["a"].to(dt)
        e = (P @ a[:h])[A.rows] + (P @ a[h:])[A.cols]
        att = torch.where(e > 0, e, ALPHA * e)
        return A.mul(P, vals=att), P, att, e
    if kind == "gcn":
        z = A.mul(X @ W)
    else:
        S, zs = X, []
        for k in range(case["K"] + 1):
            S = S if k == 0 else A.mul(S)
            zs.append(S @ W[:, k * h: (k + 1) * h])
        z = torch.cat(zs, 1)
    return z if d["b"] is None else z + d["b"].to(dt)


def _settle_kinks(case, d):
    """dY = 0 where the pre-activation lies within rounding of the kink."""
    if case["kind"] not in ("sage", "gcn", "mixhop", "gat"):
        return
    # in 64 bits, so that the choice does not depend on an order of additions
    z = _layer_z(case, d, _Adj(d["csr"], torch.float64), torch.float64)
    z = z[0] if case["kind"] == "gat" else z
    # bf16 operands: 2^-9 per operand, averaged over the sum; fp32: 2^-24
    near = (0.04 if case["mode"] == "bf16" else 1e-4) * z.square().mean(0, keepdim=True).sqrt()
    d["dY"][z.abs() < near] = 0.0


def prepare(case, seed):
    if case["kind"] == "induce":
        return _prepare_induce(case, seed)
    d = _inputs(case, seed)
    _settle_kinks(case, d)
    kind, n, f, h = case["kind"], case["n"], case["f"], case["h"]
    graph = runtime.DeviceGraph(d["csr"])
    graph.prepare()
    s = {"case": case, "graph": graph, "X": d["X"], "dY": d["dY"]}
    if kind in ("sage", "stack", "train"):
        host = lambda t: None if t is None else t.cpu().numpy()
        params = [synth.LayerParams(host(ws), host(wn), host(bs), host(bn))
                  for (ws, wn), (bs, bn) in zip(d["W"], d["b"])]
        if kind == "train":
            s["T"] = d["T"]
            s["trainer"] = runtime.Trainer(graph, params, f, host(d["W_mlp"]), False, "sgd", LR,
                                           flags=_flags(case), keep_xm=True)
        else:
            s["stack"] = runtime.SageStack(graph, params, f, flags=_flags(case))
        return s
    csr = graph.struct()
    width = d["dY"].shape[1]
    rows = lambda w: torch.empty((n, -(-w // 16) * 16), device="cuda")[:, :w]
    s.update(W=d["W"], b=d["b"], a=d.get("a"), Y=rows(width), dX=rows(f),
             dW=torch.empty((f, width), device="cuda"),
             db=torch.empty(width, device="cuda") if d["b"] is not None else None,
             da=torch.empty(2 * h, device="cuda") if kind == "gat" else None)
    lay = G.make_layer(f, h, s["X"].stride(0), s["Y"].stride(0), s["dX"].stride(0), 0,
                       _flags(case))
    if kind == "gcn":
        sizes = G.gnn_gcn_saved_bytes(csr, lay), G.gnn_gcn_workspace_bytes(csr, lay)
    elif kind == "mixhop":
        sizes = (G.gnn_mixhop_saved_bytes(csr, lay, case["K"]),
                 G.gnn_mixhop_workspace_bytes(csr, lay, case["K"]))
    else:
        sizes = G.gnn_gat_saved_bytes(csr, lay), G.gnn_gat_workspace_bytes(csr, lay)
    s["layer"] = lay
    s["saved"], s["ws"] = (torch.empty(max(b, 256), dtype=torch.uint8, device="cuda")
                           for b in sizes)
    return s


def _induce_inputs(case, seed):
    """A Kronecker graph with its nodes renumbered by a rotation (so that the
    sizes do not depend on the seed), a frontier-sampled node list, features
    and labels."""
    base = synth.kronecker_graph(case["scale"], case["deg"], 5)
    nodes = G.gnn_frontier_sample(base, case["m"], case["n"], 2.0, 0, 5, 0)
    rng = np.random.default_rng([seed, 2])
    turn = int(rng.integers(1, base.n))
    rows = np.repeat(np.arange(base.n), base.degrees())
    full = synth.full_from_pairs(base.n, (rows + turn) % base.n,
                                 (base.indices.astype(np.int64) + turn) % base.n)
    X = rng.standard_normal((full.n, case["f"]), dtype=np.float32)
    T = synth.labels(full.n, case["C"], False, rng)
    return full, X, T, np.sort((nodes + turn) % base.n).astype(np.int32)


def _prepare_induce(case, seed):
    full, X, T, nodes = _induce_inputs(case, seed)
    return {"case": case, "full": runtime.FullGraphDevice(full, X, T), "nodes": nodes}


# ------------------------------------------------------------------- run

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "induce":
        g, X, T = s["full"].induce(s["nodes"])
        return {"indptr": g.indptr, "indices": g.indices, "values": g.values,
                "values_t": g.values_t, "X": X, "T": T}
    if kind == "train":
        t = s["trainer"]
        s["graph"].prepare()
        loss = t.step(s["X"], s["T"])
        return {"loss": loss, "logits": t.xm, "weights": [w for w, _ in t.pairs]}
    if kind in ("sage", "stack"):
        st = s["stack"]
        Y = st.forward(s["X"])
        dX = st.backward(s["dY"])
        keys = ("dW_self", "dW_neigh", "db_self", "db_neigh")
        return {"Y": Y, "dX": dX, "grads": [[L[k] for k in keys] for L in st.layers]}
    csr, lay, X, Y, dY = s["graph"].struct(), s["layer"], s["X"], s["Y"], s["dY"]
    if kind == "gcn":
        G.gnn_gcn_fwd(csr, lay, X, s["W"], s["b"], Y, s["saved"], s["ws"])
        G.gnn_gcn_bwd(csr, lay, X, s["W"], Y, dY, s["saved"], s["dX"], s["dW"], s["db"], s["ws"])
    elif kind == "mixhop":
        K = case["K"]
        G.gnn_mixhop_fwd(csr, lay, K, X, s["W"], s["b"], Y, s["saved"], s["ws"])
        G.gnn_mixhop_bwd(csr, lay, K, X, s["W"], Y, dY, s["saved"], s["dX"], s["dW"], s["db"],
                         s["ws"])
    else:
        G.gnn_gat_fwd(csr, lay, X, s["W"], s["a"], ALPHA, Y, None, s["saved"], s["ws"])
        G.gnn_gat_bwd(csr, lay, X, s["W"], s["a"], ALPHA, Y, dY, s["saved"], s["dX"], s["dW"],
                      s["da"], s["ws"])
    return {"Y": Y, "dX": s["dX"], "dW": s["dW"], "db": s["db"], "da": s["da"]}


# ------------------------------------------------------------------ work

def work(case):
    """Bytes: every input read once, every output written once.  Flops: the
    dense products and the aggregations' multiply-adds of one pass."""
    if case["kind"] == "induce":
        # the rows of the sampled nodes are read (index and membership), about
        # a tenth of their entries kept
        n, f, C = 0.9 * case["n"], case["f"], case["C"]
        entries = 8.0 * case["deg"] * n
        return {"bytes": 8 * entries + 3 * 4 * 1.2 * case["deg"] * n + 8 * n * (f + C),
                "flops": 0.0}
    n, f, h, kind = case["n"], case["f"], case["h"], case["kind"]
    nnz = n * (case["deg"] + 1)
    bytes_, flops = 4.0 * (n + 1) + 12.0 * nnz, 0.0
    if kind in ("sage", "stack", "train"):
        fi = f
        for i in range(case.get("layers", 1)):
            flops += (8.0 if kind == "train" and i == 0 else 12.0) * n * fi * h
            flops += (2.0 if kind == "train" and i == 0 else 4.0) * nnz * min(fi, h)
            bytes_ += 4.0 * 4 * fi * h  # both weights read, both gradients written
            fi = 2 * h
        bytes_ += 4.0 * n * (f + 2 * h)  # X in, Y out
        if kind == "train":
            C = case["C"]
            flops += 6.0 * n * fi * C
            bytes_ += 4.0 * (2 * n * C + 2 * fi * C)
        else:
            bytes_ += 4.0 * n * (2 * h + f)  # dY in, dX out
        return {"bytes": bytes_, "flops": flops}
    width = (case["K"] + 1) * h if kind == "mixhop" else h
    hops = 2 * case["K"] * f if kind == "mixhop" else 2 * min(f, h)
    flops = 6.0 * n * f * width + 2.0 * nnz * (hops + (2 * h if kind == "gat" else 0))
    if kind == "gat":
        flops += 8.0 * n * h
    return {"bytes": bytes_ + 4.0 * (2 * n * (f + width) + 2 * f * width), "flops": flops}


def tolerance(case):
    """Measured against exact(): 32-bit sums leave 1e-7 to 1e-6, 3e-6 over
    50,000 rows, bf16 operands 2.5e-3; a stack's gradients also meet ReLU
    decisions that rounding takes the other way."""
    if case["kind"] == "induce":
        return {"rel": 1e-6}
    if case["mode"] == "bf16":
        return {"rel": 1e-2, "max": 0.2}
    if case["kind"] == "train":
        return {"rel": 1e-5, "max": 3e-4}
    if case["kind"] == "stack":
        return {"rel": 5e-3, "max": 0.9}
    return {"rel": 1e-5, "max": 3e-4}


# ----------------------------------------------------------------- exact

def exact(case, seed):
    if case["kind"] == "induce":
        return _exact_induce(case, seed)
    d = _inputs(case, seed)
    _settle_kinks(case, d)
    dt, kind, h = torch.float64, case["kind"], case["h"]
    A = _Adj(d["csr"], dt)
    X, dY = d["X"].to(dt), d["dY"].to(dt)
    if kind in ("sage", "stack", "train"):
        xs = [X]
        for i in range(len(d["W"])):
            xs.append(_layer_z(case, d, A, dt, xs[-1], i).clamp_min(0))
        up, head = dY, None
        if kind == "train":
            head = d["W_mlp"].to(dt)
            xm = (xs[-1] @ head).clamp_min(0)
            T = d["T"].to(dt)
            logp = torch.log_softmax(xm, 1)
            g = (logp.exp() - T) / case["n"] * (xm > 0)
            up = g @ head.T
        grads = []
        for i in reversed(range(len(d["W"]))):
            Gm = up * (xs[i + 1] > 0)
            Gs, Tn = Gm[:, :h], Gm[:, h:]
            Ws, Wn = (w.to(dt) for w in d["W"][i])
            if xs[i].shape[1] > h:
                AG = A.mul(Tn, True)
                dWn, back = xs[i].T @ AG, AG @ Wn.T
            else:
                dWn, back = A.mul(xs[i]).T @ Tn, A.mul(Tn @ Wn.T, True)
            grads.append([xs[i].T @ Gs, dWn] +
                         ([Gs.sum(0), Tn.sum(0)] if case["bias"] else [None, None]))
            up = Gs @ Ws.T + back
        grads.reverse()
        if kind != "train":
            return {"Y": xs[-1], "dX": up, "grads": grads}
        loss = -(T * logp).sum() / case["n"]
        ws, gs = [head], [xs[-1].T @ g]
        for w, gr in zip(d["W"], grads):
            ws += [t.to(dt) for t in w]
            gs += gr[:2]
        new = [w - LR * g for w, g in zip(ws, gs)]
        return {"loss": loss.reshape(1), "logits": xm, "weights": new}
    W = d["W"].to(dt)
    da = None
    if kind == "gat":
        z, P, att, e = _layer_z(case, d, A, dt)
        Gm = dY * (z > 0)
        dz = torch.empty_like(att)
        for k in range(0, dz.numel(), 1 << 18):
            q = slice(k, k + (1 << 18))
            dz[q] = (Gm[A.rows[q]] * P[A.cols[q]]).sum(1)
        dz = torch.where(e > 0, dz, ALPHA * dz)
        zero = torch.zeros(case["n"], dtype=dt, device="cuda")
        ds, dtt = zero.index_add(0, A.rows, dz), zero.index_add(0, A.cols, dz)
        a = d["a"].to(dt)
        dP = A.mul(Gm, True, att) + ds[:, None] * a[None, :h] + dtt[:, None] * a[None, h:]
        dW, dX, da = X.T @ dP, dP @ W.T, torch.cat([P.T @ ds, P.T @ dtt])
    else:
        z = _layer_z(case, d, A, dt)
        Gm = dY * (z > 0)
        if kind == "gcn":
            T = A.mul(Gm, True)
            dW, dX = X.T @ T, T @ W.T
        else:
            dW, dX, S = torch.empty_like(W), torch.zeros_like(X), X
            for k in range(case["K"] + 1):
                S = S if k == 0 else A.mul(S)
                cols = slice(k * h, (k + 1) * h)
                dW[:, cols] = S.T @ Gm[:, cols]
                back = Gm[:, cols] @ W[:, cols].T
                for _ in range(k):
                    back = A.mul(back, True)
                dX += back
    db = Gm.sum(0) if d["b"] is not None else None
    return {"Y": z.clamp_min(0), "dX": dX, "dW": dW, "db": db, "da": da}


def _exact_induce(case, seed):
    full, X, T, nodes = _induce_inputs(case, seed)
    pos = np.full(full.n, -1, np.int64)
    pos[nodes] = np.arange(len(nodes))
    rows = np.repeat(np.arange(full.n), full.degrees())
    keep = (pos[rows] >= 0) & (pos[full.indices] >= 0)
    r = np.concatenate([pos[rows[keep]], np.arange(len(nodes))])
    c = np.concatenate([pos[full.indices[keep]], np.arange(len(nodes))])
    order = np.lexsort((c, r))
    r, c = r[order], c[order]
    deg = np.bincount(r, minlength=len(nodes))
    indptr = np.concatenate([[0], np.cumsum(deg)])
    return {"indptr": indptr, "indices": c, "values": 1.0 / deg[r], "values_t": 1.0 / deg[c],
            "X": X[nodes].astype(np.float64), "T": T[nodes].astype(np.float64)}
