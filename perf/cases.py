"""The work that a user of the library has it do, as cases that can be timed and compared.

A case is a dict of plain values; ``kind`` selects the public entry points that ``run`` calls:

    pass       graph construction, plan and every round of a model over a small graph (harness.Pipeline)
    graph      CSR and plan from raw pairs
    transform  one dense layer
    round      one embed-and-aggregate round (transform, then aggregation)
    aggregate  one aggregation alone
    stored     the rows put into 16-bit storage, then aggregated
    attention  edge softmax in a training loop: forward in save mode, then its backward
    backward   backward of the parameter-free aggregations
    train      loss and gradients of one locally trained layer
    share      a worker's share of an edge-partitioned graph, and the rows it sends and receives

Inputs are drawn on the GPU from the seed alone: power-law graphs handed over as raw pairs (repeats and self
pairs included), normal or tf-idf-like features, Glorot parameters.
"""
import math

import numpy as np
import torch

from paper_2302_13053_amd import binding as B
from paper_2302_13053_amd import harness as Hn
from paper_2302_13053_amd import workloads as wl

SLOPE = 0.2
MANY = 1_000_000        # on-off decisions (units, scores): among more of them some lie within rounding of their edge


# ---------------------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------------------
def listed():
    reddit = dict(n=232965, pairs=58620000, exponent=2.5, max_w=23000.0, loops=False)
    products = dict(n=2449029, pairs=61920000, exponent=2.8, max_w=17500.0, loops=False)
    return [
        # a whole pass over a citation graph of a few thousand nodes (Cora-shaped): launches and latency
        dict(name="pass_sage_tiny", kind="pass", family="sage", n=2708, pairs=5429, f0=1433, hidden=64, rounds=2,
             classes=7, heads=1),
        # the next size up (PubMed-shaped): three rounds of the normalised sum with self-loops
        dict(name="pass_gcn_citation", kind="pass", family="gcn", n=19717, pairs=44338, f0=500, hidden=256, rounds=3,
             classes=3, heads=1),
        # the graph of a dense social network from its raw pairs (Reddit-shaped), paid for on every new graph
        dict(name="graph_reddit", kind="graph", **reddit),
        # the layer in front of an attention round of a large sparse graph (ogbn-products-shaped)
        dict(name="transform_products", kind="transform", n=2449029, d_in=256, d_out=256, relu=False, padded=True,
             rectified=False),
        # the final classifier of the dense graph: few output columns, an odd number of them
        dict(name="transform_classifier", kind="transform", n=232965, d_in=512, d_out=41, relu=False, padded=True,
             rectified=True),
        # first round over raw features of the dense graph: mean with self-concat, a row of 602 floats
        dict(name="mean_reddit", kind="aggregate", mode="mean", F=602, heads=1, concat=True, padded=True, **reddit),
        # last attention round of the sparse graph, heads of 47 columns (transform and aggregation)
        dict(name="round_gat_products", kind="round", mode="gat_softmax", d_in=256, F=188, heads=4, relu=False,
             concat=False, padded=True, **products),
        # an attention layer in its training loop: forward that keeps what the backward needs, and the backward
        dict(name="attention_products", kind="attention", F=256, heads=4, padded=True, **products),
        # one training step's gradients for the dense graph's hidden layer with its temporary classifier
        dict(name="train_reddit", kind="train", n=232965, d_in=1204, hidden=256, classes=41, labelled=0.66, p_drop=0.5,
             input_grad=False, padded=True),
        # the same for the smallest graph, input gradient included: latency
        dict(name="train_tiny", kind="train", n=2708, d_in=2866, hidden=64, classes=7, labelled=0.05, p_drop=0.0,
             input_grad=True, padded=True),
        # the dense graph's first round with the table in bfloat16
        dict(name="stored_reddit", kind="stored", storage="bf16", mode="mean", F=602, heads=1, concat=True,
             padded=True, **reddit),
        # worker 0 of 4 over the dense graph: its share, the rows it owes its peers, the rows it receives
        dict(name="share_reddit", kind="share", parts=4, F=602, padded=True, **reddit),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _graph(rng, most_entries=114_000_000, most_nodes=2_400_000):
    """Nodes, raw pairs and skew between the smallest and the largest graphs listed."""
    n = _log(rng, 2000, most_nodes)
    mean = math.exp(rng.uniform(math.log(4.0), math.log(500.0)))
    mean = min(mean, n / 20.0, most_entries / n)
    return dict(n=n, pairs=max(1, int(n * mean / 2)), exponent=round(rng.uniform(2.4, 3.0), 2),
                max_w=round(max(8.0, min(n / 10.0, rng.uniform(40.0, 350.0) * mean)), 1), loops=False)


def _width(rng, lo=3, hi=640):
    """A width as layers have them (multiples of 32 half the time), or any other."""
    f = _log(rng, lo, hi)
    return max(32, f // 32 * 32) if rng.random() < 0.5 else f


def _heads(rng, most=256):
    heads = rng.choice((1, 2, 4, 4, 8))
    dh = rng.choice((8, 16, 32, 64, 64, _log(rng, 3, 64)))
    return heads, heads * min(dh, most // heads)


def draw(rng):
    kind = rng.choice(("pass", "graph", "transform", "transform", "round", "aggregate", "stored", "attention",
                       "backward", "train", "train", "share"))
    padded = rng.random() < 0.75
    mode = rng.choice(("mean", "sum", "gcn_sym", "gat_softmax"))
    if kind == "pass":
        n = _log(rng, 500, 30000)
        return dict(kind=kind, family=rng.choice(("sage", "gcn", "gat")), n=n, pairs=int(n * rng.uniform(1.5, 12.0)),
                    f0=_log(rng, 20, 1500), hidden=rng.choice((32, 64, 128, 256)), rounds=rng.choice((2, 3)),
                    classes=rng.randint(2, 47), heads=rng.choice((2, 4)))
    if kind == "graph":
        return dict(kind=kind, **{**_graph(rng), "loops": rng.random() < 0.3})
    if kind == "transform":
        d_in, d_out = _log(rng, 16, 2900), _width(rng, 3, 300)
        n = _log(rng, 1000, min(2_400_000, int(1.6e11 / (d_in * d_out)), int(6.4e8 / d_in)))
        return dict(kind=kind, n=n, d_in=d_in, d_out=d_out, relu=rng.random() < 0.5, padded=padded,
                    rectified=rng.random() < 0.5)
    if kind == "train":
        d_in, hidden, classes = _log(rng, 16, 2900), rng.choice((0, 32, 64, 128, 200, 256)), rng.randint(2, 60)
        n = _log(rng, 1000, min(1_000_000, int(5.5e10 / (d_in * (hidden or classes))), int(3.2e8 / d_in)))
        return dict(kind=kind, n=n, d_in=d_in, hidden=hidden, classes=classes,
                    labelled=round(rng.choice((0.05, 0.3, 0.66, 1.0)), 2),
                    p_drop=rng.choice((0.0, 0.3, 0.5)) if hidden else 0.0, input_grad=rng.random() < 0.4, padded=padded)
    if kind == "share":
        return dict(kind=kind, parts=rng.choice((2, 3, 4, 8, 24)), F=_width(rng, 16, 602), padded=padded,
                    **_graph(rng, 60_000_000, 1_200_000))
    if kind == "attention":
        heads, F = _heads(rng)
        return dict(kind=kind, F=F, heads=heads, padded=True, **_graph(rng, int(3e10 / max(F, 128))))
    heads, F = _heads(rng) if mode == "gat_softmax" and kind != "backward" else (1, _width(rng))
    g = _graph(rng, min(114_000_000, int(4e10 / max(F, 64))))
    g["loops"] = mode == "gcn_sym"
    if kind == "backward":
        mode = "mean" if mode == "gat_softmax" else mode
        return dict(kind=kind, mode=mode, F=F, concat=rng.random() < 0.5, padded=padded, **g)
    concat = mode == "mean" and rng.random() < 0.7
    if kind == "round":
        d_in = min(_log(rng, 16, 1300), int(1.6e11 / (g["n"] * F)) or 1)
        return dict(kind=kind, mode=mode, d_in=d_in, F=F, heads=heads, relu=mode != "gat_softmax", concat=concat,
                    padded=padded, **g)
    if kind == "stored":
        return dict(kind=kind, storage=rng.choice(("bf16", "fp16")), mode=mode, F=F, heads=heads, concat=concat,
                    padded=padded, **g)
    return dict(kind=kind, mode=mode, F=F, heads=heads, concat=concat, padded=padded, **g)


# ---------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------
class _Plan:
    """A plan in memory of torch's allocator; given back with the state that holds it."""

    def __init__(self, g, split=False):
        self.memory = Hn.ws_tensor(B.retexo_plan_workspace_bytes(g.n_nodes, g.nnz, 0))
        self.graph = Hn.make_plan(g, workspace=self.memory)

    def __del__(self):
        self.graph.destroy()


class _Pipe(Hn.Pipeline):
    def __del__(self):
        self.close()


def _gen(seed, stream):
    return torch.Generator(device="cuda").manual_seed(1000003 * (int(seed) % (1 << 40)) + stream)


def _pairs(case, seed):
    """Raw undirected pairs: both ends drawn in proportion to clipped power-law weights, ids scattered."""
    n, m = case["n"], case["pairs"]
    g = _gen(seed, 0)
    base = torch.arange(1, n + 1, dtype=torch.float64, device="cuda") ** (-1.0 / (case["exponent"] - 1.0))
    lo, hi, mean = 0.0, case["max_w"] * n, 2.0 * m / n
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        if float((mid * base).clamp_(max=case["max_w"]).mean()) < mean:
            lo = mid
        else:
            hi = mid
    edge = torch.cumsum((hi * base).clamp_(max=case["max_w"]), 0)
    ids = torch.randperm(n, generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    ends = []
    for _ in range(2):
        u = torch.rand(m, generator=g, device="cuda", dtype=torch.float64).mul_(edge[-1])
        ends.append(ids[torch.searchsorted(edge, u).clamp_(max=n - 1)])
    return ends[0], ends[1]


def _ld(case, width, unit=32):
    return -(-width // unit) * unit if case["padded"] else width


def _rows(case, n, width, g, unit=32):
    """[n, ld] normal values; the columns past `width` are zero."""
    t = torch.zeros((n, _ld(case, width, unit)), dtype=torch.float32, device="cuda")
    t[:, :width].normal_(generator=g)
    return t


def _glorot(g, fan_in, fan_out, shape):
    lim = math.sqrt(6.0 / (fan_in + fan_out))
    return torch.empty(shape, dtype=torch.float32, device="cuda").uniform_(-lim, lim, generator=g)


def _bias(g, width):
    return torch.empty(width, dtype=torch.float32, device="cuda").uniform_(-0.1, 0.1, generator=g)


def _planned(case, seed):
    src, dst = _pairs(case, seed)
    g = Hn.csr_from_coo(src, dst, case["n"], case["loops"])
    g.col_idx = g.col_idx[:max(g.nnz, 1)].clone()
    return _Plan(g)


def _workload(case, seed):
    """The model over its graph, as the workload descriptions of the package state them."""
    fam, f0, hid, cls, heads = case["family"], case["f0"], case["hidden"], case["classes"], case["heads"]
    st = []
    if fam == "gat":
        width = f0
        for r in range(case["rounds"]):
            out = heads * (hid // heads if r < case["rounds"] - 1 else cls)
            st.append(wl.Stage("round", width, out, mode="gat_softmax", heads=heads))
            width = out
        st.append(wl.Stage("head_mean", width, cls, w=False, heads=heads))
    else:
        mode, concat = ("mean", True) if fam == "sage" else ("gcn_sym", False)
        st.append(wl.Stage("round", f0, f0, w=False, mode=mode, concat=concat))
        width = st[-1].out_width
        for _ in range(case["rounds"] - 1):
            st.append(wl.Stage("round", width, hid, relu=True, mode=mode, concat=concat))
            width = st[-1].out_width
        st.append(wl.Stage("transform", width, cls))
    if fam == "gcn":
        graph, args = "chung_lu", {"edges": case["pairs"], "exponent": 2.5, "max_w": 300.0}
    else:
        graph, args = "er", {"edges": case["pairs"]}
    return wl.Workload(100, "case", fam, case["n"], graph, args, fam == "gcn", f0,
                       {"sage": "bernoulli", "gcn": "tfidf", "gat": "normal"}[fam], tuple(st))


def _model(case, seed):
    w = _workload(case, seed)
    seed = int(seed) % (1 << 60)
    src, dst = wl.make_graph(w, seed)
    return w, src, dst, wl.make_features(w, ld=wl.pad_ld(w.feat_dim), seed=seed), wl.make_params(w, seed)


def _attention(g, heads, F):
    dh = F // heads
    return _glorot(g, dh, 1, (heads, dh)), _glorot(g, dh, 1, (heads, dh))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "pass":
        w, src, dst, feats, params = _model(case, seed)
        return dict(case=case, pipe=_Pipe(w, src, dst, feats, params))
    g = _gen(seed, 1)
    s = dict(case=case)
    if kind == "graph":
        src, dst = _pairs(case, seed)
        n, m, loops = case["n"], case["pairs"], case["loops"]
        cap = 2 * m + (n if loops else 0)
        i32 = lambda k: torch.empty(max(k, 1), dtype=torch.int32, device="cuda")
        s.update(src=src, dst=dst, csr_ws=Hn.ws_tensor(B.retexo_csr_workspace_bytes(m, n, loops)),
                 row_ptr=torch.empty(n + 1, dtype=torch.int64, device="cuda"), col_idx=i32(cap).zero_(),
                 plan_ws=Hn.ws_tensor(B.retexo_plan_workspace_bytes(n, cap, 0)), deg=i32(n),
                 dinv=torch.empty(n, dtype=torch.float32, device="cuda"), order=i32(n))
    elif kind == "transform":
        H = _rows(case, case["n"], case["d_in"], g)
        if case["rectified"]:
            H.relu_()
        s.update(H=H, W=_glorot(g, case["d_in"], case["d_out"], (case["d_in"], case["d_out"])),
                 b=_bias(g, case["d_out"]), out=_rows(case, case["n"], case["d_out"], g))
    elif kind == "train":
        n, d_in, hid, cls = case["n"], case["d_in"], case["hidden"], case["classes"]
        labels = torch.randint(0, cls, (n,), generator=g, device="cuda", dtype=torch.int32)
        labels[torch.rand(n, generator=g, device="cuda") > case["labelled"]] = -1
        first = hid or cls
        s.update(X=_rows(case, n, d_in, g), labels=labels, W1=_glorot(g, d_in, first, (d_in, first)),
                 b1=_bias(g, first), Wc=_glorot(g, hid, cls, (hid, cls)) if hid else None,
                 bc=_bias(g, cls) if hid else None, ws=Hn.ws_tensor(B.retexo_train_workspace_bytes(n, d_in, hid, cls)),
                 gX=_rows(case, n, d_in, g) if case["input_grad"] else None,
                 dropout=(case["p_drop"], 20230213, int(seed) % 1000) if case["p_drop"] else None)
    elif kind == "share":
        # buffers for any ownership: kept from one share to the next
        n, F, parts = case["n"], case["F"], case["parts"]
        s["plan"] = _planned(case, seed)
        s["owner"] = torch.randint(0, parts, (n,), generator=g, device="cuda", dtype=torch.int32)
        s["most"] = n, 2 * case["pairs"] + (n if case["loops"] else 0), n + 40 * math.isqrt(n)
        zero = lambda k, dtype=torch.int32: torch.zeros(k, dtype=dtype, device="cuda")
        s["arrays"] = dict(local_ids=zero(n), row_ptr=zero(n + 1, torch.int64), col_idx=zero(s["most"][1]), deg=zero(n),
                           send=zero(s["most"][2]), recv=zero(n))
        s.update(table=_rows(case, n, F, g), received=_rows(case, n, F, g),
                 to_send=zero((s["most"][2], _ld(case, F)), torch.float32),
                 ws=Hn.ws_tensor(B.retexo_partition_workspace_bytes(n, parts, s["most"][2])))
    else:
        s["plan"] = _planned(case, seed)
        n, F, heads = case["n"], case["F"], case.get("heads", 1)
        graph = s["plan"].graph
        mode = "gat_softmax" if kind == "attention" else case["mode"]
        concat = case.get("concat", False)
        width = 2 * F if concat else F
        s["a_src"], s["a_dst"] = _attention(g, heads, F) if mode == "gat_softmax" else (None, None)
        flags = (B.F_SELF_CONCAT if concat else 0) | (B.F_SAVE if kind == "attention" else 0)
        if kind == "backward":
            s["ws"] = Hn.ws_tensor(B.retexo_aggregate_backward_workspace_bytes(graph.plan, B.MODES[mode], F, 1))
            s.update(G=_rows(case, n, width, g), dZ=_rows(case, n, F, g))
            return s
        s["ws"] = Hn.ws_tensor(B.retexo_workspace_bytes(graph.plan, F, B.MODES[mode], heads, flags))
        s["out"] = _rows(case, n, width, g)
        if kind == "round":
            s.update(H=_rows(case, n, case["d_in"], g).relu_(), W=_glorot(g, case["d_in"], F, (case["d_in"], F)),
                     b=_bias(g, F))
        else:
            s["Z"] = _rows(case, n, F, g)
        if kind == "attention":
            s.update(G=_rows(case, n, F, g), dZ=_rows(case, n, F, g),
                     back_ws=Hn.ws_tensor(B.retexo_aggregate_backward_workspace_bytes(
                         graph.plan, B.MODES[mode], F, heads)))
    return s


# ---------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "pass":
        pipe = s["pipe"]
        outs = pipe.run()
        return dict(rounds=[o[:, :st.out_width] for o, st in zip(outs, pipe.wl.stages)], row_ptr=pipe.row_ptr,
                    col_idx=pipe.col_idx[:pipe.graph.nnz])
    if kind == "graph":
        g = Hn.csr_from_coo(s["src"], s["dst"], case["n"], case["loops"], s["csr_ws"], s["row_ptr"], s["col_idx"])
        Hn.make_plan(g, workspace=s["plan_ws"])
        B.check(B.retexo_plan_export(g.plan, s["deg"].data_ptr(), s["dinv"].data_ptr(), s["order"].data_ptr(),
                                     Hn._stream_ptr()), "retexo_plan_export")
        g.destroy()
        # the buffer's rest, past the entries, is never written and stays zero
        return dict(nnz=g.nnz, row_ptr=s["row_ptr"], col_idx=s["col_idx"], deg=s["deg"], dinv=s["dinv"], order=s["order"])
    if kind == "transform":
        Hn.transform(s["H"], case["d_in"], s["W"], s["b"], case["relu"], out=s["out"])
        return s["out"][:, :case["d_out"]]
    if kind == "train":
        loss, gW1, gb1, gWc, gbc = Hn.layer_grad(s["X"], case["d_in"], s["labels"], s["W1"], s["b1"], s["Wc"], s["bc"],
                                                 workspace=s["ws"], gX=s["gX"], dropout=s["dropout"])
        r = dict(loss=loss, gW1=gW1, gb1=gb1)
        if case["hidden"]:
            r.update(gWc=gWc, gbc=gbc)
        if case["input_grad"]:
            r["gX"] = s["gX"][:, :case["d_in"]]
        return r
    F = case["F"]
    graph = s["plan"].graph
    if kind == "share":
        arr = s["arrays"]
        st, sizes, send_at, recv_at = B.retexo_partition_share(
            graph.n_nodes, graph.row_ptr.data_ptr(), graph.col_idx.data_ptr(), s["owner"].data_ptr(), case["parts"], 0,
            *s["most"], arr["local_ids"].data_ptr(), arr["row_ptr"].data_ptr(), arr["col_idx"].data_ptr(),
            arr["deg"].data_ptr(), arr["send"].data_ptr(), arr["recv"].data_ptr(), s["ws"].data_ptr(), s["ws"].numel(),
            Hn._stream_ptr())
        B.check(st, "retexo_partition_share")
        _, halo, _, sends = sizes
        Hn.halo_pack(arr["send"][:sends], s["table"], F, buf=s["to_send"])
        Hn.halo_unpack(arr["recv"][:halo], s["received"], s["table"], F)
        # what lies past a share's sizes is never written
        return dict(arr, sizes=list(sizes), send_at=list(send_at), recv_at=list(recv_at), packed=s["to_send"][:, :F],
                    table=s["table"][:, :F])
    if kind == "backward":
        Hn.aggregate_backward(graph, case["mode"], F, s["G"], concat=case["concat"], dZ=s["dZ"], workspace=s["ws"])
        return s["dZ"][:, :F]
    kw = dict(heads=case["heads"], a_src=s["a_src"], a_dst=s["a_dst"], slope=SLOPE)
    if kind == "attention":
        Hn.aggregate(graph, "gat_softmax", s["Z"], F, out=s["out"], workspace=s["ws"], save=True, **kw)
        dZ, das, dad = Hn.aggregate_backward(graph, "gat_softmax", F, s["G"], Z=s["Z"], dZ=s["dZ"],
                                             workspace=s["back_ws"], saved=s["ws"], **kw)
        return dict(out=s["out"][:, :F], dZ=dZ[:, :F], da_src=das, da_dst=dad)
    width = 2 * F if case["concat"] else F
    if kind == "round":
        st = wl.Stage("round", case["d_in"], F, relu=case["relu"], mode=case["mode"], concat=case["concat"],
                      heads=case["heads"])
        Hn.round_(graph, st, s["H"], s["W"], s["b"], s["a_src"], s["a_dst"], s["out"], s["ws"], slope=SLOPE)
    elif kind == "stored":
        table = Hn.store_rows(s["Z"], F, case["storage"], ld=_ld(case, F, 64))
        Hn.aggregate_stored(graph, case["mode"], table, F, case["storage"], concat=case["concat"], out=s["out"],
                            workspace=s["ws"], **kw)
    else:
        Hn.aggregate(graph, case["mode"], s["Z"], F, concat=case["concat"], out=s["out"], workspace=s["ws"], **kw)
    return s["out"][:, :width]


# ---------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------
def work(case):
    kind, n = case["kind"], case["n"]
    if kind == "transform":
        i, o = case["d_in"], case["d_out"]
        return dict(bytes=4.0 * (n * i + i * o + n * o), flops=2.0 * n * i * o)
    if kind == "train":
        i, h, c = case["d_in"], case["hidden"], case["classes"]
        layers = i * h + h * c if h else i * c
        # forward, weight gradients, and the classifier's backward; the input gradient on request
        flops = 2.0 * n * (2 * layers + (h * c if h else 0) + (case["input_grad"] and i * (h or c)))
        return dict(bytes=4.0 * (n * i * (2 if case["input_grad"] else 1) + n + 2 * layers), flops=flops)
    entries = 2.0 * case["pairs"] + (n if case.get("loops") or case.get("family") == "gcn" else 0)
    csr = 4.0 * entries + 8.0 * n
    if kind == "graph":
        return dict(bytes=8.0 * case["pairs"] + csr + 12.0 * n, flops=0.0)
    if kind == "pass":
        by, fl = 8.0 * case["pairs"] + csr, 0.0
        for st in _workload(case, 0).stages:
            by += 4.0 * n * (st.d_in + st.out_width) + (csr if st.kind == "round" else 0.0)
            if st.w:
                by += 4.0 * st.d_in * st.d_out
                fl += 2.0 * n * st.d_in * st.d_out
            if st.kind == "round":
                fl += 2.0 * entries * st.d_out
        return dict(bytes=by, flops=fl)
    F = case["F"]
    if kind == "share":
        # the graph read, a part of it written, the rows sent and received read and written once
        rows = n * (1.0 - 1.0 / case["parts"])
        return dict(bytes=csr * (1.0 + 1.0 / case["parts"]) + 20.0 * n + 8.0 * F * (rows + n / case["parts"]), flops=0.0)
    out = (2 if case.get("concat") else 1) * F
    if kind == "backward":
        return dict(bytes=csr + 4.0 * n * (out + F), flops=2.0 * entries * F)
    if kind == "attention":
        # forward Z -> out; backward Z, G -> dZ; per entry and column: score, weighted sum, two products back
        return dict(bytes=2 * csr + 4.0 * n * F * 5, flops=10.0 * entries * F)
    gat = 2.0 * entries * F if case["mode"] == "gat_softmax" else 0.0
    if kind == "round":
        return dict(bytes=csr + 4.0 * n * (case["d_in"] + out) + 4.0 * case["d_in"] * F,
                    flops=2.0 * n * case["d_in"] * F + 2.0 * entries * F + gat)
    if kind == "stored":
        return dict(bytes=csr + n * (4.0 * F + 4.0 * F + 4.0 * out), flops=2.0 * entries * F + gat)
    return dict(bytes=csr + 4.0 * n * (F + out), flops=2.0 * entries * F + gat)


def tolerance(case):
    """About four times what the sums in float32 were seen to be off the same in 64 bits; integers and copied rows stay
    the same.  Where there are many units or scores, some are switched by rounding alone (see _train64)."""
    kind = case["kind"]
    if kind == "share":
        return "exact"
    if kind == "train" and case["n"] * case["hidden"] > MANY:
        return dict(rel=1e-4, max=0.5)
    if kind == "attention":
        if 2 * case["pairs"] * case["heads"] > MANY:
            return dict(rel=1.5e-3, max=0.9)
        return dict(rel=4e-6, max=1e-4)
    return dict(rel=4e-6, max=5e-5)


# ---------------------------------------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------------------------------------
def _csr64(src, dst, n, loops):
    """Row offsets and columns of the undirected simple graph of the raw pairs."""
    src, dst = src.long(), dst.long()
    keep = src != dst
    src, dst = src[keep], dst[keep]
    key = torch.cat([src * n + dst, dst * n + src])
    if loops:
        key = torch.cat([key, torch.arange(n, device="cuda") * (n + 1)])
    key = torch.unique(key)
    row, col = key // n, key % n
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    return rp, col, row


def _spmm64(rp, col, val, X):
    """Sum over every row's entries of val * X[col], 64-bit, in column pieces that bound the memory."""
    n = rp.numel() - 1
    out = torch.empty((n, X.shape[1]), dtype=torch.float64, device="cuda")
    if col.numel() == 0:
        return out.zero_()
    step = 64
    A = torch.sparse_csr_tensor(rp, col, val, size=(n, X.shape[0]))
    for c in range(0, X.shape[1], step):
        out[:, c:c + step] = A @ X[:, c:c + step].double().contiguous()
    return out


def _softmax64(rp, row, col, Z, heads, a_src, a_dst):
    """Per-entry scores, their softmax over each row and per-head views, 64-bit."""
    n, F = Z.shape
    dh = F // heads
    el = torch.stack([Z[:, h * dh:(h + 1) * dh].double() @ a_src[h].double() for h in range(heads)], 1)
    er = torch.stack([Z[:, h * dh:(h + 1) * dh].double() @ a_dst[h].double() for h in range(heads)], 1)
    p = el[col] + er[row]
    e = torch.where(p > 0, p, SLOPE * p)
    top = torch.full((n, heads), -math.inf, dtype=torch.float64, device="cuda")
    top.scatter_reduce_(0, row[:, None].expand(-1, heads), e, "amax")
    e = torch.exp(e - top[row])
    total = torch.zeros((n, heads), dtype=torch.float64, device="cuda").index_add_(0, row, e)
    return p, e / total[row]


def _aggregate64(mode, rp, row, col, Z, F, heads, a_src, a_dst, concat):
    n = rp.numel() - 1
    Z = Z[:, :F]
    deg = (rp[1:] - rp[:-1]).double()
    if mode == "gat_softmax":
        _, alpha = _softmax64(rp, row, col, Z, heads, a_src, a_dst)
        dh = F // heads
        out = torch.cat([_spmm64(rp, col, alpha[:, h].contiguous(), Z[:, h * dh:(h + 1) * dh]) for h in range(heads)], 1)
    elif mode == "gcn_sym":
        dinv = torch.where(deg > 0, deg.rsqrt(), torch.zeros_like(deg))
        out = _spmm64(rp, col, dinv[row] * dinv[col], Z)
    else:
        out = _spmm64(rp, col, torch.ones(col.numel(), dtype=torch.float64, device="cuda"), Z)
        if mode == "mean":
            out /= deg.clamp(min=1)[:, None]
    return torch.cat([Z.double(), out], 1) if concat else out


def _dense64(H, d_in, W, b, relu):
    Z = H[:, :d_in].double() @ W.double()
    if b is not None:
        Z += b.double()
    return Z.relu_() if relu else Z


def _mul32(a, b):
    """(high, low) 32 bits of the product of 32-bit values held in int64."""
    lo = (a & 0xFFFF) * b
    hi = (a >> 16) * b + (lo >> 16)
    return (hi >> 16) & 0xFFFFFFFF, ((hi & 0xFFFF) << 16) | (lo & 0xFFFF)


def _keep_mask(n, hidden, p, seed, number):
    """Philox-4x32-10 words of (node, unit / 4, draw number): the documented dropout mask."""
    q = -(-hidden // 4)
    c = [torch.arange(n, device="cuda")[:, None].expand(n, q).reshape(-1),
         torch.arange(q, device="cuda")[None, :].expand(n, q).reshape(-1)]
    c += [torch.full_like(c[0], number & 0xFFFFFFFF), torch.full_like(c[0], number >> 32)]
    k = [seed & 0xFFFFFFFF, seed >> 32]
    for _ in range(10):
        h0, l0 = _mul32(c[0], 0xD2511F53)
        h2, l2 = _mul32(c[2], 0xCD9E8D57)
        c = [h2 ^ c[1] ^ k[0], l2, h0 ^ c[3] ^ k[1], l0]
        k = [(k[0] + 0x9E3779B9) & 0xFFFFFFFF, (k[1] + 0xBB67AE85) & 0xFFFFFFFF]
    words = torch.stack(c, 1).reshape(n, 4 * q)[:, :hidden]
    return words >= math.floor(float(np.float32(p)) * 4294967296.0)


def _train64(s):
    case = s["case"]
    hid, n, d_in = case["hidden"], case["n"], case["d_in"]
    X, lab = s["X"][:, :d_in].double(), s["labels"].long()
    act = lab >= 0
    count = max(int(act.sum()), 1)
    pre = X @ s["W1"].double() + s["b1"].double()
    scale = 1.0
    if hid:
        mask = pre > 0
        if case["p_drop"]:
            mask &= _keep_mask(n, hid, case["p_drop"], s["dropout"][1], s["dropout"][2])
            scale = 1.0 / (1.0 - case["p_drop"])
        A = torch.where(mask, pre * scale, torch.zeros_like(pre))
        logits = A @ s["Wc"].double() + s["bc"].double()
    else:
        logits = pre
    logp = torch.log_softmax(logits, 1)
    pick = lab.clamp(min=0)[:, None]
    loss = -(logp.gather(1, pick)[:, 0] * act).sum() / count
    dL = torch.exp(logp)
    dL.scatter_add_(1, pick, torch.full_like(dL[:, :1], -1.0))
    dL *= (act.double() / count)[:, None]
    r = dict(loss=loss.reshape(1))
    if hid:
        r.update(gWc=A.T @ dL, gbc=dL.sum(0))
        dA = torch.where(mask, scale * (dL @ s["Wc"].double().T), torch.zeros_like(A))
    else:
        dA = dL
    # A unit whose sum is within rounding of zero is on or off by the rounding, and one such unit outweighs all
    # rounding of the gradients behind it: with many units these have no value to compare with.
    if hid and n * hid > MANY:
        r.update(gW1=None, gb1=None)
        if case["input_grad"]:
            r["gX"] = None
        return r
    r.update(gW1=X.T @ dA, gb1=dA.sum(0))
    if case["input_grad"]:
        r["gX"] = dA @ s["W1"].double().T
    return r


def _attention64(s):
    case = s["case"]
    F, heads = case["F"], case["heads"]
    dh = F // heads
    graph = s["plan"].graph
    n, rp = graph.n_nodes, graph.row_ptr
    col = graph.col_idx[:graph.nnz].long()
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), rp[1:] - rp[:-1])
    Z, G = s["Z"][:, :F], s["G"][:, :F]
    p, alpha = _softmax64(rp, row, col, Z, heads, s["a_src"], s["a_dst"])
    out = torch.cat([_spmm64(rp, col, alpha[:, h].contiguous(), Z[:, h * dh:(h + 1) * dh]) for h in range(heads)], 1)
    c = torch.stack([(G[:, h * dh:(h + 1) * dh].double() * out[:, h * dh:(h + 1) * dh]).sum(1) for h in range(heads)], 1)
    if col.numel() * heads > MANY:                # LeakyReLU's slope at a score within rounding of zero, as in _train64
        return dict(out=out, dZ=None, da_src=None, da_dst=None)
    dots = torch.empty_like(p)
    step = max(1, int(4e8 / F))
    for i in range(0, col.numel(), step):
        j = slice(i, i + step)
        prod = G[row[j]].double() * Z[col[j]].double()
        dots[j] = prod.reshape(-1, heads, dh).sum(2)
    # the gradient of the score before LeakyReLU
    t = alpha * torch.where(p > 0, 1.0, SLOPE) * (dots - c[row])
    del dots, p
    ddst = torch.zeros((n, heads), dtype=torch.float64, device="cuda").index_add_(0, row, t)
    dsrc = torch.zeros((n, heads), dtype=torch.float64, device="cuda").index_add_(0, col, t)
    del t
    back = torch.argsort(col * n + row)           # the graph is symmetric: entry (u, v) sits where (v, u) sorts to
    dZ = torch.cat([_spmm64(rp, col, alpha[back, h].contiguous(), G[:, h * dh:(h + 1) * dh]) for h in range(heads)], 1)
    das, dad = [], []
    for h in range(heads):
        k = slice(h * dh, (h + 1) * dh)
        dZ[:, k] += dsrc[:, h:h + 1] * s["a_src"][h].double() + ddst[:, h:h + 1] * s["a_dst"][h].double()
        das.append(Z[:, k].double().T @ dsrc[:, h])
        dad.append(Z[:, k].double().T @ ddst[:, h])
    return dict(out=out, dZ=dZ, da_src=torch.stack(das), da_dst=torch.stack(dad))


def exact(case, seed):
    kind = case["kind"]
    if kind == "share":
        return None                               # integers and copied rows
    if kind == "graph":
        src, dst = _pairs(case, seed)
        rp, _, _ = _csr64(src, dst, case["n"], case["loops"])
        deg = (rp[1:] - rp[:-1]).double()
        return dict(nnz=None, row_ptr=None, col_idx=None, deg=None, order=None,
                    dinv=torch.where(deg > 0, deg.rsqrt(), torch.zeros_like(deg)))
    if kind == "pass":
        w, src, dst, feats, params = _model(case, seed)
        rp, col, row = _csr64(torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), w.n_nodes, w.self_loops)
        H = torch.from_numpy(feats).cuda().double()
        outs = []
        for st, p in zip(w.stages, params):
            W, b, a_src, a_dst = (None if a is None else torch.from_numpy(a).cuda() for a in (p.W, p.b, p.a_src, p.a_dst))
            if st.kind == "head_mean":
                H = H[:, :st.d_in].reshape(-1, st.heads, st.d_out).mean(1)
            else:
                Z = H if W is None else _dense64(H, st.d_in, W, b, st.relu)
                H = Z if st.kind == "transform" else _aggregate64(st.mode, rp, row, col, Z, st.d_out, st.heads, a_src,
                                                                  a_dst, st.concat)
            outs.append(H)
        return dict(rounds=outs, row_ptr=None, col_idx=None)
    s = prepare(case, seed)
    if kind == "transform":
        return _dense64(s["H"], case["d_in"], s["W"], s["b"], case["relu"])
    if kind == "train":
        return _train64(s)
    if kind == "attention":
        return _attention64(s)
    graph = s["plan"].graph
    F, rp, col = case["F"], graph.row_ptr, graph.col_idx[:graph.nnz].long()
    row = torch.repeat_interleave(torch.arange(graph.n_nodes, device="cuda"), rp[1:] - rp[:-1])
    if kind == "backward":
        G = s["G"]
        own, G = (G[:, :F].double(), G[:, F:2 * F]) if case["concat"] else (0.0, G[:, :F])
        if case["mode"] == "mean":                # symmetric graph: the transposed mean sums the scaled rows
            G = G.double() / (rp[1:] - rp[:-1]).clamp(min=1)[:, None]
        return own + _aggregate64("gcn_sym" if case["mode"] == "gcn_sym" else "sum", rp, row, col, G, F, 1, None, None,
                                  False)
    if kind == "round":
        Z = _dense64(s["H"], case["d_in"], s["W"], s["b"], case["relu"])
    elif kind == "stored":
        Z = s["Z"][:, :F].to({"bf16": torch.bfloat16, "fp16": torch.float16}[case["storage"]]).double()
    else:
        Z = s["Z"]
    return _aggregate64(case["mode"], rp, row, col, Z, F, case["heads"], s["a_src"], s["a_dst"], case["concat"])
