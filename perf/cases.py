"""The work that programs have this library do, as cases to be timed.

Every case goes through the public entry points (``gcn``, ``model``): whole
training epochs and an inference pass of the two-layer GCN, single layers
forward and backward over a CSR and a dense A_hat, the loss, the decoder of
the graph auto-encoder, the construction of A_hat and the optimiser.  Sizes
and graph families are those of ``inputs.SPECS``, of the model-size sweep
(``inputs.table1_workload``) and of the tests.

Graphs and inputs are drawn on the GPU from the case's seed.  ``exact``
recomputes each case in float64 with plain torch and numpy.
"""
import math

import numpy as np
import torch

from paper_2010_12635_amd import gcn as G
from paper_2010_12635_amd import inputs as I
from paper_2010_12635_amd.model import AdamConfig, DeviceGraph, GCN2

PRECS = {"f32": G.GCN_F32, "f16": G.GCN_F16, "bf16": G.GCN_BF16}
BYTES = {"f32": 4, "f16": 2, "bf16": 2}
LOSS_SCALE = 65536.0
DEV = "cuda"


def listed():
    return [
        # Smallest training epoch: 2048 papers with 512 sparse features, 7
        # classes, 140 labelled vertices (the citation-network setup).  Bound
        # by launches and latency.
        {"name": "epoch_er2k_f16", "kind": "epoch", "graph": "er", "n": 2048, "m": 4, "adj": "csr", "index": "i32",
         "f_in": 512, "hidden": 16, "classes": 7, "n_mask": 140, "dropout": 0.5, "prec": "f16"},
        # An epoch as the paper runs it: every tensor dense, A_hat included
        # (16384 vertices in 32 blocks, 500 features).
        {"name": "epoch_sbm16k_dense_f16", "kind": "epoch", "graph": "sbm", "n": 16384, "m": 4, "adj": "dense",
         "index": "i32", "f_in": 500, "hidden": 64, "classes": 32, "n_mask": 0, "dropout": 0.5, "prec": "f16"},
        # Inference of a trained model on a power-law graph (evaluation mode,
        # logits of every vertex), bfloat16.
        {"name": "infer_rmat17_bf16", "kind": "infer", "graph": "rmat", "n": 1 << 17, "m": 16, "adj": "csr",
         "index": "i32", "f_in": 256, "hidden": 256, "classes": 64, "n_mask": 0, "dropout": 0.5, "prec": "bf16"},
        # Hidden layer of the largest training workload, forward with ReLU
        # and dropout: 2M vertices, 65.6M entries, 64-bit row pointers.
        {"name": "fwd_rmat21_f16", "kind": "fwd", "graph": "rmat", "n": 1 << 21, "m": 16, "adj": "csr",
         "index": "i64", "f_in": 128, "f_out": 128, "dropout": 0.5, "prec": "f16"},
        # Output layer backward in full precision on the paper's graph
        # family: 40 classes, gradients of W, of both biases and of the
        # hidden layer.
        {"name": "bwd_ba200k_f32", "kind": "bwd", "graph": "ba", "n": 200000, "m": 8, "adj": "csr", "index": "i32",
         "f_in": 128, "f_out": 40, "dropout": 0.5, "prec": "f32"},
        # Softmax cross-entropy of the largest workload and its gradient.
        {"name": "loss_rmat21_f16", "kind": "loss", "n": 1 << 21, "classes": 64, "n_mask": 0, "prec": "f16"},
        # The largest point of the model-size sweep: featureless input, dense
        # A_hat, 2048 hidden units, forward with ReLU and dropout.
        {"name": "fwd_featureless_n32768_d2048_f16", "kind": "fwd", "graph": "ba", "n": 32768, "m": 8,
         "adj": "dense", "index": "i32", "f_in": 0, "f_out": 2048, "dropout": 0.5, "prec": "f16"},
        # A middle point of the sweep, backward (dW1 = A_hat dZ).
        {"name": "bwd_featureless_n8192_d512_bf16", "kind": "bwd", "graph": "ba", "n": 8192, "m": 8,
         "adj": "dense", "index": "i32", "f_in": 0, "f_out": 512, "dropout": 0.5, "prec": "bf16"},
        # A dense layer of odd size in full precision.
        {"name": "fwd_dense_n6001_f32", "kind": "fwd", "graph": "ba", "n": 6001, "m": 8, "adj": "dense",
         "index": "i32", "f_in": 130, "f_out": 48, "dropout": 0.5, "prec": "f32"},
        # Link prediction, one epoch of the decoder: 2^20 training edges and
        # 2^20 random pairs drawn, scored, and their gradient into Z.
        {"name": "pairs_rmat17_f16", "kind": "pairs", "n": 1 << 17, "f_out": 64, "n_pos": 1 << 20,
         "n_neg": 1 << 20, "prec": "f16"},
        # Construction of A_hat from an edge list, with its schedule: what
        # every program does first with a graph.
        {"name": "graph_rmat18_f16", "kind": "graph", "graph": "rmat", "n": 1 << 18, "m": 16, "index": "i32",
         "prec": "f16"},
        # Adam with dynamic loss scaling on the weights of a featureless
        # model (16384 vertices x 512 hidden units).
        {"name": "adam_n16384_d512_f16", "kind": "adam", "count": 16384 * 512 + 512 + 512 * 16 + 16,
         "prec": "f16"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["epoch", "epoch", "infer", "fwd", "fwd", "bwd", "bwd", "loss", "pairs", "graph", "adam"])
    prec = rng.choice(["f16", "f16", "bf16", "f32"])
    if kind == "loss":
        n = _log_int(rng, 2000, 1 << 20)
        return {"kind": kind, "n": n, "classes": rng.randint(2, 96), "n_mask": rng.choice([0, n // 10]), "prec": prec}
    if kind == "adam":
        return {"kind": kind, "count": _log_int(rng, 2000, 8 << 20), "prec": prec}
    if kind == "pairs":
        return {"kind": kind, "n": _log_int(rng, 2000, 1 << 17), "f_out": rng.randint(8, 128 if prec != "f32" else 96),
                "n_pos": _log_int(rng, 1 << 13, 1 << 20), "n_neg": _log_int(rng, 1 << 13, 1 << 20), "prec": prec}
    if kind == "graph":
        g = rng.choice(["rmat", "ba"])
        n = 1 << rng.randint(11, 17) if g == "rmat" else _log_int(rng, 2000, 200000)
        return {"kind": kind, "graph": g, "n": n, "m": rng.randint(4, 16), "index": rng.choice(["i32", "i64"]),
                "prec": prec}
    c = {"kind": kind, "adj": rng.choice(["csr", "csr", "dense"]), "index": rng.choice(["i32", "i64"]),
         "dropout": rng.choice([0.0, 0.5, 0.3]), "prec": prec}
    if c["adj"] == "dense":
        c.update(graph="ba", n=_log_int(rng, 1100, 12000), m=8, index="i32")
    else:
        c["graph"] = rng.choice(["er", "ba", "rmat"])
        c["n"] = 1 << rng.randint(11, 18) if c["graph"] == "rmat" else _log_int(rng, 1100, 200000)
        c["m"] = rng.randint(4, 16)
    if kind in ("epoch", "infer"):
        c.update(f_in=_log_int(rng, 16, 512), hidden=_log_int(rng, 8, 256), classes=rng.randint(2, 64),
                 n_mask=rng.choice([0, c["n"] // 10]))
    elif c["adj"] == "dense" and rng.random() < 0.5:
        c.update(f_in=0, f_out=_log_int(rng, 64, 1024))                  # featureless input
    else:
        c.update(f_in=_log_int(rng, 16, 512), f_out=_log_int(rng, 8, 256))
    return c


# ------------------------------------------------------------------ inputs ----

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _edges(case, seed):
    """Raw undirected edge samples (repeats and self-loops possible)."""
    n, m, gen = case["n"], case["m"], _gen(seed)
    if case["graph"] == "rmat":
        return I.rmat_graph_device(n.bit_length() - 1, m, 0.57, 0.19, 0.19, seed, DEV)
    if case["graph"] == "er":
        e = m * n
        return (torch.randint(0, n, (e,), generator=gen, device=DEV, dtype=torch.int32),
                torch.randint(0, n, (e,), generator=gen, device=DEV, dtype=torch.int32))
    if case["graph"] == "sbm":       # 32 equal blocks, p_in = 0.01, p_out = 0.0002
        b, s = 32, n // 32
        e_in, e_out = int(0.01 * b * s * (s - 1) / 2), int(0.0002 * b * (b - 1) / 2 * s * s)
        blk = torch.randint(0, b, (e_in,), generator=gen, device=DEV)
        u, v = (blk * s + torch.randint(0, s, (e_in,), generator=gen, device=DEV) for _ in range(2))
        p, q = (torch.randint(0, n, (e_out,), generator=gen, device=DEV) for _ in range(2))
        return torch.cat([u, p]).int(), torch.cat([v, q]).int()
    # Barabasi-Albert: edge k links vertex m + k / m to a uniform choice among
    # the endpoints so far (which is a choice in proportion to degree); the
    # choices that fall on an earlier edge's target follow it back
    e = m * (n - m)
    k = torch.arange(e, device=DEV)
    src = m + k // m
    before = 2 * m * torch.clamp(src - m, min=1)
    pick = (torch.rand(e, generator=gen, device=DEV, dtype=torch.float64) * before).long().clamp_(max=2 * e - 1)
    pick = torch.where(src == m, -1 - (k % m), pick)        # the first vertex links to the m seeds
    while True:
        odd = (pick >= 0) & (pick % 2 == 1)
        if not bool(odd.any()):
            break
        pick = torch.where(odd, pick[torch.where(odd, pick // 2, torch.zeros_like(pick))], pick)
    dst = torch.where(pick < 0, -1 - pick, m + torch.clamp(pick, min=0) // 2 // m)
    return src.int(), dst.int()


def _dtype(case):
    return G.torch_dtype(PRECS[case["prec"]])


def _padded(n, f, gen, dtype, scale=1.0):
    x = torch.zeros((n, (f + 7) // 8 * 8), dtype=dtype, device=DEV)
    step = 1 << 20
    for lo in range(0, n, step):
        hi = min(n, lo + step)
        x[lo:hi, :f] = (torch.randn((hi - lo, f), generator=gen, device=DEV) * scale).to(dtype)
    return x


def _glorot(f_in, f_out, gen):
    return (torch.rand((f_in, f_out), generator=gen, device=DEV) * 2 - 1) * math.sqrt(6.0 / (f_in + f_out))


def _mask(n, k, gen):
    if not k:
        return torch.ones(n, dtype=torch.uint8, device=DEV)
    m = torch.zeros(n, dtype=torch.uint8, device=DEV)
    m[torch.randperm(n, generator=gen, device=DEV)[:k]] = 1
    return m


def _inputs(case, seed):
    """Everything drawn for a case but its graph, in the layout and type that the calls take."""
    kind, dt, gen = case["kind"], _dtype(case) if "prec" in case else None, _gen(seed * 1000003 + 17)
    n = case.get("n")
    if kind in ("epoch", "infer"):
        f, h, c = case["f_in"], case["hidden"], case["classes"]
        if case["graph"] == "er":      # bag-of-words features, 1 % of them set
            x = _padded(n, f, gen, dt, 0.0)
            x[:, :f] = (torch.rand((n, f), generator=gen, device=DEV)
                        * (torch.rand((n, f), generator=gen, device=DEV) < 0.01)).to(dt)
        else:
            x = _padded(n, f, gen, dt)
        return dict(X=x, W1=_glorot(f, h, gen), W2=_glorot(h, c, gen),
                    labels=torch.randint(0, c, (n,), generator=gen, device=DEV, dtype=torch.int32),
                    mask=_mask(n, case["n_mask"], gen))
    if kind in ("fwd", "bwd"):
        ident = case["f_in"] == 0
        f_in, f_out = (n if ident else case["f_in"]), case["f_out"]
        w = torch.zeros((f_in, (f_out + 7) // 8 * 8), dtype=dt, device=DEV)
        w[:, :f_out] = _glorot(f_in, f_out, gen).to(dt)
        d = dict(W=w, b=torch.zeros(w.shape[1], device=DEV), H=None if ident else _padded(n, f_in, gen, dt))
        d["b"][:f_out] = torch.randn(f_out, generator=gen, device=DEV) * 0.1
        if kind == "bwd":              # loss-scaled gradients; the hidden layer below went through ReLU and dropout
            d["dZ"] = _padded(n, f_out, gen, dt, LOSS_SCALE / n if case["prec"] != "f32" else 1.0 / n)
            if not ident:
                h = d["H"]
                h.copy_(torch.where(torch.rand(h.shape, generator=gen, device=DEV) < case["dropout"],
                                    torch.zeros_like(h), torch.clamp(h, min=0)))
        return d
    if kind == "loss":
        c = case["classes"]
        return dict(Z=_padded(n, c, gen, dt, 1.5),
                    labels=torch.randint(0, c, (n,), generator=gen, device=DEV, dtype=torch.int32),
                    mask=_mask(n, case["n_mask"], gen))
    if kind == "pairs":
        e = case["n_pos"] * 2
        # endpoints of the training edges are skewed like those of an R-MAT graph
        eu, ev = (torch.clamp((torch.rand(e, generator=gen, device=DEV, dtype=torch.float64) ** 3 * n).int(), max=n - 1)
                  for _ in range(2))
        perm = torch.randperm(n, generator=gen, device=DEV).int()
        return dict(Z=_padded(n, case["f_out"], gen, dt, 0.35), eu=perm[eu.long()], ev=perm[ev.long()])
    if kind == "adam":
        k = case["count"]
        r = lambda s: torch.randn(k, generator=gen, device=DEV) * s    # noqa: E731
        return dict(master=r(0.02), grad=r(1e-4 * LOSS_SCALE), m=r(1e-5), v=r(1e-4) ** 2)
    return {}


def _graph(case, seed, prec):
    src, dst = _edges(case, seed)
    return DeviceGraph(case["n"], src, dst, prec=prec, index=G.GCN_I64 if case["index"] == "i64" else G.GCN_I32,
                       dense=case.get("adj") == "dense")


def prepare(case, seed):
    kind, x = case["kind"], _inputs(case, seed)
    prec = PRECS[case["prec"]]
    dt = _dtype(case)
    st = dict(case=case, seed=seed, prec=prec, **x)
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    if kind in ("epoch", "infer"):
        g = _graph(case, seed, prec)
        m = GCN2(g, x["X"], x["labels"], x["mask"], x["W1"].cpu().numpy(), x["W2"].cpu().numpy(), prec=prec,
                 dropout=case["dropout"], seed=seed, loss_scale=LOSS_SCALE, adam=AdamConfig())
        # as after some hundred epochs: second moments that have settled
        m.v.fill_(1e-6)
        m.scaler[1] = 200
        m.scaler[2] = 200
        st["model"] = m
    elif kind in ("fwd", "bwd"):
        g = _graph(case, seed, prec)
        ident = case["f_in"] == 0
        f_in, f_out = (case["n"] if ident else case["f_in"]), case["f_out"]
        ld_in, ld = (f_in + 7) // 8 * 8, x["W"].shape[1]
        L = G.GcnLayer(f_in, f_out, ld_in, ld, G.GCN_ACT_RELU, case["dropout"], 0, 1 if ident else 0)
        ws = torch.empty(G.gcn_layer_workspace_size(g.adj, L, prec), dtype=torch.uint8, device=DEV)
        e = lambda w: torch.empty((case["n"], w), dtype=dt, device=DEV)    # noqa: E731
        st.update(g=g, L=L, ws=ws, flag=flag, S=e(ld))
        if kind == "fwd":
            st["out"] = e(ld)
        else:
            st.update(dW=torch.empty((f_in, ld), device=DEV), db=torch.empty(ld, device=DEV),
                      dZb=None if ident else e(ld_in), dbb=None if ident else torch.empty(ld_in, device=DEV))
    elif kind == "loss":
        n, c = case["n"], case["classes"]
        st.update(ws=torch.empty(G.gcn_loss_workspace_size(n, c), dtype=torch.uint8, device=DEV), flag=flag,
                  scale=torch.full((1,), LOSS_SCALE if case["prec"] != "f32" else 1.0, device=DEV),
                  loss=torch.zeros(1, device=DEV), dZ=torch.empty_like(x["Z"]),
                  cs=torch.empty(x["Z"].shape[1], device=DEV), nc=torch.zeros(1, dtype=torch.int32, device=DEV),
                  n_mask=case["n_mask"] or n)
    elif kind == "pairs":
        k, n = case["n_pos"] + case["n_neg"], case["n"]
        nb = max(G.gcn_pair_loss_workspace_size(k), G.gcn_pair_backward_workspace_size(n, k, case["f_out"]))
        i = lambda: torch.empty(k, dtype=torch.int32, device=DEV)    # noqa: E731
        st.update(ws=torch.empty(nb, dtype=torch.uint8, device=DEV), flag=flag, pu=i(), pv=i(),
                  g=torch.empty(k, device=DEV), sc=torch.empty(k, device=DEV), loss=torch.zeros(1, device=DEV),
                  scale=torch.full((1,), LOSS_SCALE if case["prec"] != "f32" else 1.0, device=DEV),
                  dZ=torch.empty_like(x["Z"]))
    elif kind == "graph":
        st["src"], st["dst"] = _edges(case, seed)
        n, e, idx = case["n"], st["src"].numel(), torch.int64 if case["index"] == "i64" else torch.int32
        nb = G.gcn_schedule_size(n, 2 * e + n)
        st.update(ws=torch.empty(G.gcn_normalize_workspace_size(n, e), dtype=torch.uint8, device=DEV),
                  sched=torch.empty(nb, dtype=torch.uint8, device=DEV),
                  rowptr=torch.zeros(n + 1, dtype=idx, device=DEV),
                  colidx=torch.zeros(2 * e + n, dtype=torch.int32, device=DEV),
                  deg=torch.zeros(n, dtype=torch.int32, device=DEV), dinv=torch.zeros(n, device=DEV),
                  values=torch.zeros(2 * e + n, dtype=dt, device=DEV))
    elif kind == "adam":
        s = torch.zeros(4, dtype=torch.int32, device=DEV)
        s.view(torch.float32)[0] = LOSS_SCALE
        s[1] = 200
        s[2] = 200
        st.update(state=s, flag=flag, working=x["master"].to(dt), cfg=AdamConfig().c())
    return st


def run(st):
    case, prec = st["case"], st["prec"]
    kind = case["kind"]
    if kind == "epoch":
        m = st["model"]
        m.step(0)
        return {"logits": m.Z2[:, :m.C], "loss": m.loss, "grad": m.grad, "weights": m.master}
    if kind == "infer":
        m = st["model"]
        m.forward(0, training=False)
        return {"logits": m.Z2[:, :m.C]}
    if kind == "fwd":
        G.gcn_layer_fwd(st["g"].adj, st["L"], prec, True, st["H"], st["W"], st["b"], st["seed"], 0,
                        None if st["H"] is None else st["S"], st["out"], st["flag"], st["ws"])
        return {"out": st["out"][:, :case["f_out"]]}
    if kind == "bwd":
        ident = st["H"] is None
        G.gcn_layer_bwd(st["g"].adj, st["L"], prec, st["H"], st["W"], st["dZ"],
                        G.GCN_ACT_NONE if ident else G.GCN_ACT_RELU, 0.0 if ident else case["dropout"], st["dW"],
                        st["db"], st["dZb"], st["S"], st["flag"], st["ws"], dbias_below=st["dbb"])
        f, fi = case["f_out"], case["f_in"]
        d = {"dW": st["dW"][:, :f], "db": st["db"][:f], "GS": st["S"][:, :f]}
        if not ident:
            d.update(dZb=st["dZb"][:, :fi], dbb=st["dbb"][:fi])
        return d
    if kind == "loss":
        n, c = case["n"], case["classes"]
        G.gcn_loss(n, c, st["Z"].shape[1], prec, st["Z"], st["labels"], st["mask"], st["n_mask"], st["scale"],
                   st["loss"], st["dZ"], st["nc"], st["flag"], st["ws"], dlogits_colsum=st["cs"])
        return {"loss": st["loss"], "dZ": st["dZ"][:, :c], "db": st["cs"][:c], "correct": st["nc"]}
    if kind == "pairs":
        n, f, ld = case["n"], case["f_out"], st["Z"].shape[1]
        np_, nn = case["n_pos"], case["n_neg"]
        G.gcn_sample_pairs(n, st["eu"], st["ev"], np_, nn, st["seed"], 0, st["pu"], st["pv"])
        G.gcn_pair_loss(n, f, ld, prec, st["Z"], st["pu"], st["pv"], np_, nn, st["scale"], st["loss"], st["sc"],
                        st["g"], st["flag"], st["ws"])
        G.gcn_pair_backward(n, f, ld, prec, st["Z"], st["pu"], st["pv"], np_ + nn, st["g"], st["dZ"], ld,
                            st["flag"], st["ws"])
        return {"u": st["pu"], "v": st["pv"], "loss": st["loss"], "scores": st["sc"], "g": st["g"],
                "dZ": st["dZ"][:, :f]}
    if kind == "graph":
        idx = G.GCN_I64 if case["index"] == "i64" else G.GCN_I32
        a = G.GcnAdj()
        a.n = case["n"]
        a.nnz = G.gcn_normalize(case["n"], st["src"], st["dst"], idx, st["rowptr"], st["colidx"], st["deg"],
                                st["dinv"], prec, st["values"], None, 0, st["ws"])
        a.format, a.index, a.value_prec = G.GCN_CSR, idx, prec
        a.rowptr, a.colidx = st["rowptr"].data_ptr(), st["colidx"].data_ptr()
        a.values, a.dinv = st["values"].data_ptr(), st["dinv"].data_ptr()
        G.gcn_schedule(a, st["sched"])
        return {"nnz": a.nnz, "rowptr": st["rowptr"], "colidx": st["colidx"], "deg": st["deg"], "dinv": st["dinv"],
                "values": st["values"]}
    G.gcn_optimizer_step(case["count"], st["master"], st["grad"], st["m"], st["v"], st["working"], prec, st["cfg"],
                         st["state"], st["flag"])
    return {"master": st["master"], "m": st["m"], "v": st["v"], "working": st["working"],
            "scale": st["state"].view(torch.float32)[:1], "steps": st["state"][1:]}


# ----------------------------------------------------------- sizes and bounds ----

def _nnz(case):
    """Entries of A_hat, to a few per cent (repeats of an R-MAT graph collapse)."""
    n, m = case["n"], case["m"]
    if case["graph"] == "rmat":
        return n + int(2 * m * n * 0.9)
    if case["graph"] == "sbm":
        return n + int(0.01 * n * (n / 32) + 0.0002 * n * n)
    return n + 2 * m * n


def _agg(case, F):
    """(bytes, flops) of one product A_hat X, X with F columns."""
    n, s = case["n"], BYTES[case["prec"]]
    if case["adj"] == "dense":
        return s * n * n + 2 * s * n * F, 2 * n * n * F
    rp = 8 if case["index"] == "i64" else 4
    return (n + 1) * rp + _nnz(case) * (4 + s) + 2 * s * n * F, 2 * _nnz(case) * F


def work(case):
    kind, s = case["kind"], BYTES[case["prec"]]
    if kind == "adam":
        return {"bytes": case["count"] * (16 + 12 + s), "flops": case["count"] * 15}
    n = case["n"]
    if kind == "loss":
        return {"bytes": 2 * s * n * case["classes"] + 5 * n, "flops": 8 * n * case["classes"]}
    if kind == "pairs":
        k, f = case["n_pos"] + case["n_neg"], case["f_out"]
        return {"bytes": 2 * s * n * f + 16 * k, "flops": 6 * k * f}
    if kind == "graph":
        e, nz = case["m"] * n, _nnz(case)
        return {"bytes": 8 * e + n * (12 if case["index"] == "i64" else 8) + 4 * n + nz * (4 + s), "flops": 2 * nz}
    if kind in ("epoch", "infer"):
        f, h, c = case["f_in"], case["hidden"], case["classes"]
        a1, a2 = _agg(case, h), _agg(case, c)
        t = 2 * n * h * (f + c)
        b, fl = a1[0] + a2[0] + s * n * (f + 2 * h + c), a1[1] + a2[1] + t
        if kind == "epoch":
            b += a1[0] + a2[0] + s * n * (2 * c) + s * n * (c + h + h) + s * n * (f + h) + 28 * h * (f + c)
            fl += a1[1] + a2[1] + t + 2 * n * h * c
        return {"bytes": b, "flops": fl}
    f = case["f_out"]
    b, fl = _agg(case, f)
    if case["f_in"]:
        b, fl = b + s * n * (case["f_in"] + f), fl + 2 * n * case["f_in"] * f
        if kind == "bwd":
            b, fl = b + s * n * case["f_in"], fl + 2 * n * case["f_in"] * f
    elif kind == "bwd":
        b += 4 * n * f
    return {"bytes": b, "flops": fl}


def tolerance(case):
    """About four times the error against exact() on MI355X (in whole epochs that of the gradients)."""
    kind, prec = case["kind"], case["prec"]
    if kind == "graph":
        return "exact"
    if kind in ("epoch", "infer"):
        return {"f32": {"rel": 2e-5}, "f16": {"rel": 1.6e-2, "max": 0.6}, "bf16": {"rel": 3e-2, "max": 0.9}}[prec]
    if kind == "adam":
        return {"rel": {"f32": 2e-6, "f16": 1e-3, "bf16": 8e-3}[prec]}
    # the column sums of the loss gradient add terms of both signs that nearly cancel
    return {"rel": {"f32": 2e-5 if kind == "loss" else 4e-6, "f16": 1.5e-3, "bf16": 1e-2}[prec]}


# ------------------------------------------------------------------- float64 ----

def _csr64(case, seed):
    """(rowptr, rows, cols, values) of A_hat, float64."""
    src, dst = _edges(case, seed)
    n = case["n"]
    u, v = src.long(), dst.long()
    keep = u != v
    u, v = u[keep], v[keep]
    d = torch.arange(n, device=DEV)
    key = torch.unique(torch.cat([u * n + v, v * n + u, d * n + d]))
    r, c = key // n, key % n
    deg = torch.bincount(r, minlength=n)
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rp[1:] = deg.cumsum(0)
    di = 1.0 / deg.double().sqrt()
    return rp, r, c, di[r] * di[c], deg, di


def _agg64(a, X):
    _, r, c, v = a[:4]
    out = torch.zeros_like(X)
    step = max(1, (1 << 28) // X.shape[1])
    for lo in range(0, r.numel(), step):
        hi = min(r.numel(), lo + step)
        out.index_add_(0, r[lo:hi], X[c[lo:hi]] * v[lo:hi, None])
    return out


def _philox4x32(ctr, key):
    """Philox-4x32-10 on int64 tensors (or numbers) of 32-bit words."""
    M = 0xFFFFFFFF
    x0, x1, x2, x3 = ctr
    k0, k1 = key

    def mul(a, b):
        t = a * (b & 0xFFFF)
        u = a * (b >> 16) + (t >> 16)
        return u >> 16, ((u & 0xFFFF) << 16) | (t & 0xFFFF)

    for _ in range(10):
        h0, l0 = mul(0xD2511F53, x0)
        h1, l1 = mul(0xCD9E8D57, x2)
        x0, x1, x2, x3 = h1 ^ x1 ^ k0, l1, h0 ^ x3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return x0, x1, x2, x3


def _keep(n, f, p, seed, layer=0, epoch=0):
    """Dropout factors (0 or 1 / (1 - p)) of an n x f layer output."""
    if p <= 0:
        return 1.0
    b = torch.arange((n * f + 3) // 4, device=DEV)
    z = torch.zeros_like(b)
    w = torch.stack(_philox4x32((b & 0xFFFFFFFF, b >> 32, z + epoch, z + layer),
                                (seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF)), 1).reshape(-1)[:n * f]
    p = float(np.float32(p))
    return (w >= int(math.floor(p * 4294967296.0))).double().view(n, f) / (1.0 - p)


def _softmax_ce(Z, labels, mask, k, scale):
    lse = torch.logsumexp(Z, 1)
    y = labels.long()
    w = mask.double() / k
    loss = ((lse - Z.gather(1, y[:, None])[:, 0]) * w).sum()
    d = torch.exp(Z - lse[:, None])
    d.scatter_add_(1, y[:, None], torch.full_like(Z[:, :1], -1.0))
    return loss, d * (w * scale)[:, None]


def _adam64(w, g, m, v, t, scale, c):
    g = g / scale
    m = c.beta1 * m + (1 - c.beta1) * g
    v = c.beta2 * v + (1 - c.beta2) * g * g
    return w - c.lr * (m / (1 - c.beta1 ** t)) / ((v / (1 - c.beta2 ** t)).sqrt() + c.eps), m, v


def _flat(parts):
    out = []
    for p in parts:
        p = p if p.dim() == 2 else p[None]
        q = torch.zeros((p.shape[0], (p.shape[1] + 7) // 8 * 8), dtype=torch.float64, device=DEV)
        q[:, :p.shape[1]] = p
        out.append(q.reshape(-1))
    return torch.cat(out)


def _pairs64(case, x, seed):
    """Philox-4x64-10 draws of the decoder's pairs."""
    n, np_, k = case["n"], case["n_pos"], case["n_pos"] + case["n_neg"]
    M32 = np.uint64(0xFFFFFFFF)
    s32 = np.uint64(32)

    def mul(a, b):
        a = np.uint64(a)
        al, ah, bl, bh = a & M32, a >> s32, b & M32, b >> s32
        t = al * bl
        m1 = ah * bl + (t >> s32)
        m2 = al * bh + (m1 & M32)
        return ah * bh + (m1 >> s32) + (m2 >> s32), a * b

    z = np.zeros(k, np.uint64)
    x0, x1, x2, x3 = np.arange(k, dtype=np.uint64), z, z, z
    k0, k1 = seed & (2 ** 64 - 1), 0x50414952
    with np.errstate(over="ignore"):
        for _ in range(10):
            h0, l0 = mul(0xD2E7470EE14C6C93, x0)
            h1, l1 = mul(0xCA5A826395121157, x2)
            x0, x1, x2, x3 = h1 ^ x1 ^ np.uint64(k0), l1, h0 ^ x3 ^ np.uint64(k1), l0
            k0, k1 = (k0 + 0x9E3779B97F4A7C15) % 2 ** 64, (k1 + 0xBB67AE8584CAA73B) % 2 ** 64
        e = torch.from_numpy((x0[:np_] % np.uint64(x["eu"].numel())).astype(np.int64)).to(DEV)
        un = x0[np_:] % np.uint64(n)
        vn = (un + np.uint64(1) + x1[np_:] % np.uint64(n - 1)) % np.uint64(n)
    t = lambda a: torch.from_numpy(a.astype(np.int64)).to(DEV)    # noqa: E731
    return torch.cat([x["eu"][e].long(), t(un)]), torch.cat([x["ev"][e].long(), t(vn)])


def exact(case, seed):
    kind, x = case["kind"], _inputs(case, seed)
    scale = LOSS_SCALE if case["prec"] != "f32" else 1.0
    if kind == "adam":
        c = AdamConfig()
        f = lambda v: float(np.float32(v))    # noqa: E731  (the constants cross the C interface as binary32)
        c = AdamConfig(lr=f(c.lr), beta1=f(c.beta1), beta2=f(c.beta2), eps=f(c.eps))
        w, m, v = _adam64(x["master"].double(), x["grad"].double(), x["m"].double(), x["v"].double(), 201,
                          LOSS_SCALE, c)
        return {"master": w, "m": m, "v": v, "working": w, "scale": torch.tensor([LOSS_SCALE], dtype=torch.float64),
                "steps": None}
    if kind == "loss":
        loss, d = _softmax_ce(x["Z"][:, :case["classes"]].double(), x["labels"], x["mask"],
                              case["n_mask"] or case["n"], scale)
        # the column sums are those of the stored (rounded) gradient: sums of
        # both signs that almost cancel have no value of their own here
        return {"loss": loss.reshape(1), "dZ": d, "db": None, "correct": None}
    if kind == "pairs":
        u, v = _pairs64(case, x, seed)
        Z = x["Z"][:, :case["f_out"]].double()
        y = (torch.arange(u.numel(), device=DEV) < case["n_pos"]).double()
        s = (Z[u] * Z[v]).sum(1)
        g = scale * (torch.sigmoid(s) - y) / u.numel()
        d = torch.zeros_like(Z)
        d.index_add_(0, u, Z[v] * g[:, None])
        d.index_add_(0, v, Z[u] * g[:, None])
        loss = (torch.nn.functional.softplus(s) - y * s).mean()
        return {"u": u.int(), "v": v.int(), "loss": loss.reshape(1), "scores": s, "g": g, "dZ": d}
    a = _csr64(case, seed)
    if kind == "graph":
        cap = 2 * _edges(case, seed)[0].numel() + case["n"]
        pad = lambda t: torch.nn.functional.pad(t, (0, cap - t.numel()))    # noqa: E731
        return {"nnz": a[2].numel(), "rowptr": a[0], "colidx": pad(a[2].int()), "deg": a[4].int(), "dinv": a[5],
                "values": pad(a[3])}
    n, p = case["n"], case["dropout"]
    if kind in ("fwd", "bwd"):
        f = case["f_out"]
        W = x["W"][:, :f].double()
        H = None if x["H"] is None else x["H"][:, :case["f_in"]].double()
        if kind == "fwd":
            out = _agg64(a, W if H is None else H @ W).add_(x["b"][:f].double()).clamp_(min=0)
            return {"out": out * _keep(n, f, p, seed)}
        dz = x["dZ"][:, :f].double()
        gs = _agg64(a, dz)
        d = {"dW": gs if H is None else H.T @ gs, "db": dz.sum(0), "GS": gs}
        if H is not None:
            db = (gs @ W.T) * (H > 0) / (1.0 - float(np.float32(p)))
            d.update(dZb=db, dbb=db.sum(0))
        return d
    dt = _dtype(case)
    W1, W2 = x["W1"].to(dt).double(), x["W2"].to(dt).double()
    X = x["X"][:, :case["f_in"]].double()
    train = kind == "epoch"
    k = _keep(n, case["hidden"], p, seed) if train else 1.0
    H1 = _agg64(a, X @ W1).clamp_(min=0) * k
    Z2 = _agg64(a, H1 @ W2)
    if not train:
        return {"logits": Z2}
    loss, dz2 = _softmax_ce(Z2, x["labels"], x["mask"], case["n_mask"] or n, scale)
    g2 = _agg64(a, dz2)
    dz1 = (g2 @ W2.T) * (H1 > 0) / (1.0 - float(np.float32(p)))
    grad = _flat([X.T @ _agg64(a, dz1), dz1.sum(0), H1.T @ g2, dz2.sum(0)])
    master = _flat([x["W1"].double(), torch.zeros(case["hidden"], device=DEV).double(), x["W2"].double(),
                    torch.zeros(case["classes"], device=DEV).double()])
    w, _, _ = _adam64(master, grad, torch.zeros_like(grad), torch.full_like(grad, 1e-6), 201, scale, AdamConfig())
    return {"logits": Z2, "loss": loss.reshape(1), "grad": grad, "weights": w}
