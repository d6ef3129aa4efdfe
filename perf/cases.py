"""The work whose speed counts: whole models and layer chains of the library, called through
its public binding, over the range of graphs that it serves.

A case is one inference pass (or, for the `new_graph` kind, the build of an adjacency and one
inference pass on it) on a synthetic graph of a stated size and shape.  Everything a program
keeps between calls -- the context, the adjacency, packed weights, activation buffers -- is made
by prepare(); run() makes the library calls of one pass and nothing else.
"""
from __future__ import annotations

import ctypes
import math

import torch

from paper_2305_02522_amd import binding as B

# What each kind stands for:
#   gcn        binary GCN on float features, layer calls (BinaryGNN.forward) or, on small
#              graphs, the one-launch model (BinaryGNN.forward_fused)
#   sage       binary GraphSAGE with sum aggregation (BinaryGNN.forward)
#   gcn_full   two-layer GCN whose products are binary and whose aggregation over
#              D^-1/2 A D^-1/2 is in float (the full-precision-aggregation recipe)
#   gcn_norm   two-layer binary GCN with the normalised adjacency, int8 features packed first
#   sage_mean  two-layer binary GraphSAGE with the mean aggregator (r = 1/deg)
#   merge      mean aggregation of float rows, merged with the node's own row by ADD and
#              binarized: a GraphSAGE layer that keeps its activations in float
#   new_graph  a graph that arrives with the request (inductive inference, sampled
#              subgraphs): edge list -> adjacency -> two-layer binary GCN


def listed():
    return [
        # citation graph of the smallest usual size: latency and launches are all there is
        dict(name="gcn small one launch", kind="gcn", graph="sbm", n=2708, deg=3.9, k0=1433,
             hidden=64, classes=7, layers=2, one_launch=True),
        # a larger citation graph through the ordinary layer calls
        dict(name="gcn small layer calls", kind="gcn", graph="sbm", n=19717, deg=4.5, k0=500,
             hidden=64, classes=3, layers=2, one_launch=False),
        # hub-heavy R-MAT graph, three layers, 256 channels: products and aggregations alike
        dict(name="gcn rmat 3 layers", kind="gcn", graph="rmat", n=1 << 17, deg=32.0, k0=512,
             hidden=256, classes=40, layers=3, one_launch=False),
        # sparse power-law graph with wide ragged features (500), GraphSAGE
        dict(name="sage sparse", kind="sage", graph="chunglu", n=89250, deg=10.0, k0=500,
             hidden=256, classes=7, layers=2),
        # dense power-law graph (mean degree 492), ragged widths 602 and 41: the benchmark's
        # own workload
        dict(name="gcn dense", kind="gcn", graph="chunglu", n=232965, deg=492.0, k0=602,
             hidden=128, classes=41, layers=2, one_launch=False),
        # the largest graph, three layers, 100 input features and 47 classes
        dict(name="sage large", kind="sage", graph="chunglu", n=2449029, deg=50.0, k0=100,
             hidden=256, classes=47, layers=3),
        # float aggregation on the dense graph
        dict(name="gcn full dense", kind="gcn_full", graph="chunglu", n=232965, deg=492.0, k0=602,
             hidden=128, classes=41, layers=2),
        # normalised binary GCN on the R-MAT graph, int8 features
        dict(name="gcn norm rmat", kind="gcn_norm", graph="rmat", n=1 << 17, deg=32.0, k0=512,
             hidden=256, classes=40, layers=2),
        # mean aggregator on the sparse graph
        dict(name="sage mean sparse", kind="sage_mean", graph="chunglu", n=89250, deg=10.0,
             k0=500, hidden=256, classes=7, layers=2),
        # float rows of an odd width on a graph of middling density
        dict(name="merge float rows", kind="merge", graph="chunglu", n=300001, deg=50.0, k0=100,
             hidden=100, classes=100, layers=1),
        # a sampled subgraph per request: the build's fixed costs
        dict(name="new graph small", kind="new_graph", graph="chunglu", n=10007, deg=10.0, k0=500,
             hidden=256, classes=7, layers=2),
        # a whole new dense graph: the build's sorts
        dict(name="new graph dense", kind="new_graph", graph="chunglu", n=232965, deg=492.0,
             k0=602, hidden=128, classes=41, layers=2),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["gcn", "gcn", "sage", "gcn_full", "gcn_norm", "sage_mean", "merge",
                       "new_graph"])
    n_hi = {"gcn": 600e3, "sage": 2.4e6, "gcn_full": 400e3, "gcn_norm": 400e3,
            "sage_mean": 600e3, "merge": 800e3, "new_graph": 300e3}[kind]
    n = int(_log(rng, 2.5e3, n_hi))
    nnz_hi = {"sage": 110e6, "gcn": 100e6, "gcn_full": 60e6, "gcn_norm": 40e6, "sage_mean": 40e6,
              "merge": 40e6, "new_graph": 60e6}[kind]
    deg = round(_log(rng, 3.0, min(500.0, n / 8.0, nnz_hi / n)), 1)
    graph = rng.choice(["sbm", "chunglu", "chunglu", "rmat"])
    if graph == "rmat":
        n = 1 << max(11, int(math.log2(n)))
        deg = min(deg, 64.0)
    # features no larger than the largest listed feature matrix
    k0 = int(_log(rng, 24, max(32.0, min(1500.0, 230e6 / n))))
    hidden = rng.choice([32, 64, 100, 128, 192, 256, int(_log(rng, 20, 256))])
    classes = rng.choice([3, 7, 10, 40, 41, 47, int(_log(rng, 2, 100))])
    layers = rng.choice([2, 2, 3]) if kind in ("gcn", "sage") else 2
    c = dict(kind=kind, graph=graph, n=n, deg=deg, k0=k0, hidden=hidden, classes=classes,
             layers=layers)
    if kind == "gcn":
        c["one_launch"] = layers == 2 and n <= 20000 and rng.random() < 0.5
    if kind == "merge":
        c["k0"] = c["hidden"] = c["classes"] = int(_log(rng, 16, 256))
        c["layers"] = 1
    return c


# ---------------------------------------------------------------- graphs


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 2654435761 % (1 << 40) + 17)
    return g


def _edges(case, g):
    """Raw undirected pairs (duplicates left in), int32 on the GPU, ids in random order."""
    n, m = int(case["n"]), int(case["n"] * case["deg"] / 2)
    u = lambda k: torch.rand(k, generator=g, device="cuda")  # noqa: E731
    if case["graph"] == "rmat":  # (a, b, c) = (.57, .19, .19)
        src = torch.zeros(m, dtype=torch.int32, device="cuda")
        dst = torch.zeros(m, dtype=torch.int32, device="cuda")
        for _ in range(n.bit_length() - 1):
            r = u(m)
            src = src * 2 + (r >= 0.76)
            dst = dst * 2 + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    elif case["graph"] == "sbm":  # seven blocks, 80 % of the pairs inside one
        src = torch.randint(0, n, (m,), generator=g, device="cuda")
        size = max(1, n // 7)
        near = (src // size) * size + torch.randint(0, size, (m,), generator=g, device="cuda")
        far = torch.randint(0, n, (m,), generator=g, device="cuda")
        dst = torch.where(u(m) < 0.8, near.clamp(max=n - 1), far)
    else:  # Chung-Lu power law, exponent 2.1, expected degrees capped at sqrt(n deg)
        total = n * float(case["deg"])
        cap = math.sqrt(total)
        raw = (torch.arange(n, dtype=torch.float64, device="cuda") + 10.0) ** (-1.0 / 1.1)
        lo, hi = 0.0, total / float(raw[-1])
        for _ in range(40):
            mid = 0.5 * (lo + hi)
            lo, hi = (mid, hi) if float((raw * mid).clamp(max=cap).sum()) < total else (lo, mid)
        cdf = torch.cumsum((raw * hi).clamp(max=cap), 0)
        cdf /= cdf[-1].clone()
        pick = lambda: torch.searchsorted(  # noqa: E731
            cdf, torch.rand(m, generator=g, device="cuda", dtype=torch.float64), right=True
        ).clamp(max=n - 1)
        src, dst = pick(), pick()
    perm = torch.randperm(n, generator=g, device="cuda").to(torch.int32)
    src, dst = perm[src.long()], perm[dst.long()]
    if case["graph"] != "rmat":
        keep = src != dst
        src, dst = src[keep], dst[keep]
    return src.contiguous(), dst.contiguous()


_hip = None


def _degrees(adj):
    """The handle's degree array as a tensor."""
    global _hip
    if _hip is None:
        _hip = ctypes.CDLL("libamdhip64.so")
        _hip.hipMemcpy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
    deg = torch.empty(adj.n, dtype=torch.int32, device="cuda")
    if _hip.hipMemcpy(deg.data_ptr(), adj.csr_pointers()[2], 4 * adj.n, 3) != 0:
        raise RuntimeError("hipMemcpy of the degrees failed")
    return deg


# ---------------------------------------------------------------- states


class _Layer:
    def __init__(self, w, t_mm, t_agg, alpha):
        self.w, self.t_mm, self.t_agg, self.alpha = w, t_mm, t_agg, alpha


def _dims(case):
    return [case["k0"]] + [case["hidden"]] * (case["layers"] - 1) + [case["classes"]]


def _params(case, g, model):
    dims, out = _dims(case), []
    thr = lambda k: torch.randint(-4, 5, (k,), generator=g, device="cuda").to(torch.int32)  # noqa: E731
    for i in range(len(dims) - 1):
        k, m, last = dims[i], dims[i + 1], i == len(dims) - 2
        kt = k if model == "gcn" else 2 * k
        w = (torch.randint(0, 2, (kt, m), generator=g, device="cuda") * 2 - 1).to(torch.int8)
        t_mm = None if last else thr(m)
        t_agg = thr(k) if model == "sage" else (None if last else thr(m))
        alpha = torch.rand(m, generator=g, device="cuda") + 0.5 if last else None
        out.append(_Layer(w, t_mm, t_agg, alpha))
    return out


def _packed(ctx, w):
    k, m = w.shape
    wb = torch.zeros((m, B.words(k)), dtype=torch.int64, device="cuda")
    B.pack_weights_i8(ctx, w, k, m, m, wb, B.words(k))
    return wb


def _packed_cat(ctx, w, k):
    """Weights of a [self | neighbour] row: both halves start at a word."""
    m, kw = w.shape[1], B.words(k)
    wb = torch.zeros((m, 2 * kw), dtype=torch.int64, device="cuda")
    B.pack_weights_i8(ctx, w, k, m, m, wb, 2 * kw)
    B.pack_weights_i8(ctx, w[k:], k, m, m, wb[:, kw:], 2 * kw)
    return wb


def prepare(case, seed):
    g = _gen(seed)
    kind, n = case["kind"], int(case["n"])
    k0, hid, m = case["k0"], case["hidden"], case["classes"]
    ctx = B.Context(0)
    s = dict(case=case, ctx=ctx)
    src, dst = _edges(case, g)
    flags = B.ADJ_SYMMETRIZE | (0 if kind in ("sage", "sage_mean", "merge") else B.ADJ_ADD_SELF_LOOPS)
    if case["graph"] == "sbm" and kind == "gcn":
        # bag-of-words features: few positive entries
        x = torch.rand((n, k0), generator=g, device="cuda").lt(0.013).float() * 2 - 1
    else:
        x = torch.randn((n, k0), generator=g, device="cuda")
    i64 = lambda *sh: torch.zeros(sh, dtype=torch.int64, device="cuda")  # noqa: E731
    f32 = lambda *sh: torch.empty(sh, dtype=torch.float32, device="cuda")  # noqa: E731
    if kind == "new_graph":
        p = _params(case, g, "gcn")
        s.update(src=src, dst=dst, flags=flags, x=x, p=p, w1=_packed(ctx, p[0].w),
                 w2=_packed(ctx, p[1].w), tmp=i64(n, B.words(hid)), h=i64(n, B.words(hid)),
                 z=torch.empty((n, m), dtype=torch.int32, device="cuda"), adj=None)
        torch.cuda.synchronize()
        return s
    adj = B.adj_build(ctx, src, dst, src.numel(), n, flags)
    del src, dst
    s["adj"] = adj
    if kind in ("gcn", "sage"):
        s.update(x=x, net=B.BinaryGNN(ctx, kind, adj, _dims(case), _params(case, g, kind)))
        return s
    deg = _degrees(adj).to(torch.float64).clamp(min=1.0)
    B.ctx_reserve(ctx, B.adj_workspace_bytes(ctx, adj, min(2048, max(k0, hid, m)), max(hid, m)))
    if kind == "merge":
        s.update(x=x, r=(1.0 / deg).float(), y=f32(n, k0), out=i64(n, B.words(k0)),
                 tau=0.3 * torch.randn(k0, generator=g, device="cuda"))
    elif kind == "sage_mean":
        p = _params(case, g, "sage")
        s.update(x=x, r=(1.0 / deg).float(), p=p, w1=_packed_cat(ctx, p[0].w, k0),
                 w2=_packed_cat(ctx, p[1].w, hid), c0=i64(n, 2 * B.words(k0)),
                 c1=i64(n, 2 * B.words(hid)), logits=f32(n, m),
                 tau0=0.3 * torch.randn(k0, generator=g, device="cuda"),
                 tau1=0.3 * torch.randn(hid, generator=g, device="cuda"))
    else:  # gcn_full, gcn_norm
        p = _params(case, g, "gcn")
        dinv = (deg ** -0.5).float()
        s.update(p=p, d=dinv, w1=_packed(ctx, p[0].w), w2=_packed(ctx, p[1].w),
                 a1=torch.rand(hid, generator=g, device="cuda") + 0.5, tmp2=f32(n, m),
                 tau=torch.randn(hid, generator=g, device="cuda"), h=i64(n, B.words(hid)),
                 logits=f32(n, m))
        if kind == "gcn_full":
            s.update(x=x, tmp1=f32(n, hid))
        else:
            x8 = torch.randint(-127, 128, (n, k0), generator=g, device="cuda").to(torch.int8)
            s.update(x8=x8, xb=i64(n, B.words(k0)), tmp1=i64(n, B.words(hid)))
    torch.cuda.synchronize()
    return s


# ---------------------------------------------------------------- one pass


def run(s):
    c = s["case"]
    kind, ctx = c["kind"], s["ctx"]
    if kind in ("gcn", "sage"):
        net = s["net"]
        if c.get("one_launch") and net.fused_applies:
            return net.forward_fused(s["x"])
        return net.forward(s["x"])
    n, k0, hid, m = int(c["n"]), c["k0"], c["hidden"], c["classes"]
    kw, hw = B.words(k0), B.words(hid)
    if kind == "new_graph":
        if s["adj"] is not None:
            s["adj"].close()  # the previous request's graph
        adj = s["adj"] = B.adj_build(ctx, s["src"], s["dst"], s["src"].numel(), n, s["flags"])
        B.ctx_reserve(ctx, B.adj_workspace_bytes(ctx, adj, hid, m))
        p, logits = s["p"], torch.empty((n, m), dtype=torch.float32, device="cuda")
        B.gcn_layer_f32(ctx, adj, s["x"], k0, k0, None, s["w1"], hid, kw, p[0].t_mm, p[0].t_agg,
                        s["tmp"], s["h"], hw)
        B.gcn_out_layer(ctx, adj, s["h"], hw, hid, hw, s["w2"], m, hw, p[1].alpha, s["z"], logits,
                        m)
        return {"nnz": adj.nnz, "max_degree": adj.max_degree, "h": s["h"], "logits": logits}
    adj = s["adj"]
    if kind == "merge":
        B.spmm_f32(ctx, adj, s["x"], False, k0, k0, s["r"], None, B.EPI_SCALE_F32, None, s["y"], k0)
        B.add(ctx, s["x"], False, k0, s["y"], False, k0, n, k0, B.EPI_THRESH_BITS, s["tau"],
              s["out"], kw)
        return s["y"], s["out"]
    p = s["p"]
    if kind == "sage_mean":
        B.pack_f32(ctx, s["x"], n, k0, k0, None, s["c0"], 2 * kw)
        B.sage_layer_weighted(ctx, adj, s["c0"], k0, s["w1"], hid, 2 * kw, s["r"], None, s["tau0"],
                              p[0].t_mm, s["c1"], 2 * hw)
        B.spmm_f32(ctx, adj, s["c1"], True, hid, 2 * hw, s["r"], None, B.EPI_THRESH_BITS,
                   s["tau1"], s["c1"][:, hw:], 2 * hw)
        B.bgemm(ctx, s["c1"], n, 2 * hw, 2 * hid, 2 * hw, s["w2"], m, 2 * hw, B.EPI_SCALE_F32,
                None, p[1].alpha, s["logits"], m)
        return s["c1"], s["logits"]
    if kind == "gcn_full":
        B.gcn_layer_full_f32(ctx, adj, s["x"], k0, k0, None, s["w1"], hid, kw, s["a1"], s["d"],
                             s["d"], s["tau"], s["tmp1"], s["h"], hw)
    else:
        B.pack_i8(ctx, s["x8"], n, k0, k0, s["xb"], kw)
        B.gcn_layer_weighted(ctx, adj, s["xb"], kw, k0, kw, s["w1"], hid, kw, p[0].t_mm, s["d"],
                             s["d"], s["tau"], s["tmp1"], s["h"], hw)
    B.gcn_out_layer_weighted(ctx, adj, s["h"], hw, hid, hw, s["w2"], m, hw, p[1].alpha, s["d"],
                             s["d"], s["tmp2"], s["logits"], m)
    return s["h"], s["logits"]


# ---------------------------------------------------------------- what a pass needs


def work(case):
    """Bytes: features, weights and (per aggregation, since layers depend on each other) the
    column ids at 4 bytes and row offsets, activations in bits written and read once per step,
    logits.  Operations: two per product term, one per aggregated channel of an edge."""
    kind, n, dims = case["kind"], int(case["n"]), _dims(case)
    # what is left of the drawn pairs once duplicates have gone
    nnz = n * case["deg"] * (0.92 if case["graph"] == "rmat" else 0.97)
    if kind not in ("sage", "sage_mean", "merge"):
        nnz += n
    csr = 4 * nnz + 4 * n
    if kind == "merge":
        c = case["k0"]
        return dict(bytes=csr + 4 * n * c * 2 + 4 * n + n * c / 8, flops=(2 * nnz + 2 * n) * c)
    by = n * case["k0"] * (1 if kind == "gcn_norm" else 4) + 4 * n * case["classes"]
    fl = 0
    if kind == "new_graph":
        by += 4 * n * case["deg"] + csr  # the edge list in, the adjacency out
    for i in range(len(dims) - 1):
        k, m = dims[i], dims[i + 1]
        two = 2 if kind in ("sage", "sage_mean") else 1
        by += csr + two * k * m / 8 + (n * k / 8 if i else 0) + (n * m / 8 if i < len(dims) - 2 else 0)
        fl += 2 * n * two * k * m + nnz * (k if two == 2 else m)
    return dict(bytes=by, flops=fl)


def tolerance(case):
    """Every sum is an exact integer, or a float sum whose order and roundings the entry point
    states (neighbours in stored order, no fused multiply-add): nothing may differ."""
    return "exact"
