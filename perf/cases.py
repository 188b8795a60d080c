"""What the framework's speed is judged by: whole passes through its public entry points, the way a program that
trains or serves a heterogeneous graph network calls them (runner.Model, binding.Context).

A case names a graph family (the shapes this repository's tests and benchmark use), what is done with a mini-batch of
it, and the sizes:

  family    "academic"     4 vertex types, 8 relations (4 and their reverses), up to 1.1M vertices, ~20M edges
            "types10"      10 vertex types of ragged feature widths, 30 relations
            "relations104" 7 types, 104 relations, 7.3k vertices in all; "relations108": 108 relations, 1.9M vertices
            "pair"         2 types, 3 relations, a few hundred vertices
  layer     "mean" (R-GCN: mean aggregation, sum fusion) or "attention" (R-GAT with semantic-attention fusion)
  mode      "step"     feature merge, all layers forward, loss, all layers backward; index arrays already built
            "forward"  feature merge and all layers forward (inference)
            "train"    a step and the Adam update of all weights and of the embedding rows the mini-batch read
            "lists"    a step whose index arrays are built in the call from the sampler's COO lists
            "sampled"  inference on given targets: sampling, index build, feature merge and forward in the call
  fanout    neighbours kept per vertex and relation, hop nearest the targets first

Mini-batches are drawn by layer-wise neighbour sampling from graphs with heavy-tailed degrees (endpoints weighted by
min(Zipf(2.1), 1e4)), features are N(0,1) or, for learnable embeddings, N(0,0.1), weights are Glorot-uniform."""
import math
import random

import numpy as np
import torch

from paper_2408_08490_amd import binding
from paper_2408_08490_amd.runner import Model

FAMILIES = ("academic", "types10", "relations104", "relations108", "pair")


def listed():
    def case(name, family, mode, dtype, targets, fanout, hidden, out, layer="mean", heads=1):
        return dict(name=name, family=family, mode=mode, layer=layer, dtype=dtype, targets=targets, fanout=fanout,
                    hidden=hidden, out=out, heads=heads)
    return [
        # a tiny graph, one layer: what a call costs when there is next to nothing to compute
        case("pair-f32-64", "pair", "step", "f32", 64, "5", 0, 16),
        # small knowledge graph with many relations, each of them tiny: launches and tables
        case("relations104-f32-128", "relations104", "step", "f32", 128, "10,10", 64, 32),
        # large knowledge graph with many relations
        case("relations108-bf16-1024", "relations108", "step", "bf16", 1024, "10,10", 128, 64),
        # many vertex types of ragged widths
        case("types10-f32-512", "types10", "step", "f32", 512, "10,10", 128, 128),
        # node classification on the academic graph in fp32, 349 classes
        case("academic-f32-1024", "academic", "step", "f32", 1024, "25,20", 256, 349),
        # the same in bf16 with large mini-batches: the headline workload of bench.py
        case("academic-bf16-4096", "academic", "step", "bf16", 4096, "25,20", 512, 349),
        # the same with the parameter update: a training step
        case("academic-bf16-4096-train", "academic", "train", "bf16", 4096, "25,20", 512, 349),
        # inference, an ordinary batch with nothing round about its sizes
        case("academic-bf16-1001-forward", "academic", "forward", "bf16", 1001, "15,10", 264, 100),
        # a training step that starts from the sampler's lists
        case("academic-bf16-1024-lists", "academic", "lists", "bf16", 1024, "25,20", 512, 349),
        # answering a request: sample around the targets, build, infer
        case("academic-bf16-256-sampled", "academic", "sampled", "bf16", 256, "15,10", 256, 349),
        # graph attention, small, in fp32
        case("attention-f32-200", "academic", "step", "f32", 200, "10,5", 128, 64, "attention", 4),
        # graph attention, three layers, bf16 storage: the largest
        case("attention-bf16-2048", "academic", "step", "bf16", 2048, "15,10,5", 256, 256, "attention", 8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    layer = "attention" if rng.random() < 0.25 else "mean"
    family = rng.choice(("academic", "academic", "academic", "types10", "relations104", "relations108", "pair"))
    if layer == "attention" and family == "pair":
        family = "academic"
    mode = rng.choice(("step", "step", "step", "forward"))
    if family == "academic" and layer == "mean":
        mode = rng.choice(("step", "step", "forward", "train", "lists", "sampled"))
    dtype = rng.choice(("bf16", "f32"))
    most = {"academic": 4096, "types10": 512, "relations104": 256, "relations108": 1024, "pair": 150}[family]
    if layer == "attention":
        most = {"academic": 1024, "types10": 256, "relations104": 256, "relations108": 512}[family]
    most = {"lists": 1024, "sampled": 512}.get(mode, most)
    targets = _log_int(rng, 24, most)
    hops = 1 if family == "pair" else rng.choice((2, 2, 2, 3)) if layer == "attention" else 2
    top = {"academic": 20, "types10": 10, "relations104": 10, "relations108": 10, "pair": 8}[family]
    fan = [rng.randint(3, top) for _ in range(hops)]
    if hops == 3:
        fan = [min(f, m) for f, m in zip(fan, (12, 8, 5))]
    if layer == "attention":
        heads = rng.choice((1, 2, 4, 8))
        hidden = rng.choice((64, 128, 256))
        out = rng.choice((64, 128))
    else:
        heads = 1
        hidden = 8 * _log_int(rng, 4, 64)
        out = rng.randint(2, 349)
    return dict(family=family, mode=mode, layer=layer, dtype=dtype, targets=targets, fanout=",".join(map(str, fan)),
                hidden=hidden, out=out, heads=heads)


# ---- graphs -----------------------------------------------------------------------------------------------------
class _Schema:
    """Vertex counts, feature widths and relations of a family: part of the case, not of the seed."""

    def __init__(self, family):
        rng = np.random.default_rng(len(family) * 1000 + 11)
        reverses, self.skew = True, True
        if family == "academic":
            self.nodes, self.feat = [736_000, 1_130_000, 8_700, 60_000], [128] * 4
            pairs = [(1, 0, 7_100_000), (0, 0, 5_400_000), (0, 3, 7_500_000), (1, 2, 1_000_000)]
            self.target, self.learnable = 0, [0, 1, 1, 1]       # type 0 carries fixed features
        elif family == "pair":
            self.nodes, self.feat = [200, 300], [16, 32]
            pairs, reverses, self.skew = [(0, 1, 1500), (1, 0, 1500), (1, 1, 1500)], False, False
            self.target, self.learnable = 1, None
        elif family == "types10":
            self.nodes = [int(x) for x in np.exp(rng.uniform(np.log(5e3), np.log(5e5), 10))]
            self.feat = [int(x) for x in rng.choice([32, 64, 128, 256, 384], 10)]
            pairs = [(int(a), int(b), 2_000_000) for a, b in zip(rng.integers(0, 10, 30), rng.integers(0, 10, 30))]
            reverses, self.learnable = False, None
            self.target = int(np.argmax(np.bincount([d for _, d, _ in pairs], minlength=10)))
        else:
            n_pairs, total, edges, width = (52, 7_300, 24_000, 64) if family == "relations104" else (54, 1_900_000, 2_850_000, 128)
            self.nodes = [max(8, int(total * x)) for x in (0.42, 0.25, 0.15, 0.1, 0.05, 0.02, 0.01)]
            self.feat = [width] * 7
            share = np.exp(rng.normal(0.0, 1.8, n_pairs))
            pairs = [(int(rng.integers(0, 7)), int(rng.integers(0, 7)), max(4, int(edges * x))) for x in share / share.sum()]
            self.target, self.learnable = 0, None
        self.pairs, self.rels = pairs, []                        # rels: (source type, destination type, pair, reversed)
        for i, (s, d, _) in enumerate(pairs):
            self.rels.append((s, d, i, False))
            if reverses:
                self.rels.append((d, s, i, True))
        self.num_types, self.num_rels = len(self.nodes), len(self.rels)
        self.rel_src, self.rel_dst = [r[0] for r in self.rels], [r[1] for r in self.rels]


class _Graph:
    """Endpoint weights of every relation; edges are drawn from them, for a mini-batch or all at once."""

    def __init__(self, sch, seed, dev):
        self.sch, self.dev = sch, dev
        self.gen = torch.Generator(dev).manual_seed(seed * 7919 + 12345)
        self.w, self.cum = [], []
        for s, d, _ in sch.pairs:
            ws, wd = (self._weights(sch.nodes[t]) for t in (s, d))
            self.w.append((ws, wd))
            self.cum.append((ws.cumsum(0), wd.cumsum(0)))

    def _weights(self, n):
        if not self.sch.skew:
            return torch.ones(n, device=self.dev, dtype=torch.float64)
        u = self.rand(n).clamp_(min=1e-9)
        return u.pow_(-1.0 / 1.1).floor_().clamp_(1.0, 1e4)

    def rand(self, n):
        return torch.rand(n, generator=self.gen, device=self.dev, dtype=torch.float64)

    def _pick(self, cum, n):
        return torch.searchsorted(cum, self.rand(n) * cum[-1], right=True).clamp_(max=cum.numel() - 1)

    def neighbours(self, r, rows, fanout):
        """(position in `rows`, source vertex) of the edges kept for the destination vertices `rows` of relation r."""
        s, d, i, rev = self.sch.rels[r]
        w = self.w[i][0 if rev else 1]
        lam = w[rows] * (self.sch.pairs[i][2] / float(w.sum()))
        deg = torch.poisson(lam, generator=self.gen).clamp_(max=fanout).long()
        row = torch.repeat_interleave(torch.arange(rows.numel(), device=self.dev), deg)
        u = self._pick(self.cum[i][1 if rev else 0], row.numel())
        key = torch.unique(row * self.sch.nodes[s] + u)
        return key // self.sch.nodes[s], key % self.sch.nodes[s]

    def targets(self, n):
        return torch.randperm(self.sch.nodes[self.sch.target], generator=self.gen, device=self.dev)[:n]

    def all_edges(self):
        """Per relation (in_indptr, in_nbr) on the host."""
        indptr, nbr = [None] * self.sch.num_rels, [None] * self.sch.num_rels
        for i, (s, d, e) in enumerate(self.sch.pairs):
            src, dst = self._pick(self.cum[i][0], e), self._pick(self.cum[i][1], e)
            for r, (a, b, j, rev) in enumerate(self.sch.rels):
                if j != i:
                    continue
                u, v = (dst, src) if rev else (src, dst)
                key = torch.unique(v * self.sch.nodes[a] + u)
                count = torch.bincount(key // self.sch.nodes[a], minlength=self.sch.nodes[b])
                indptr[r] = torch.nn.functional.pad(count.cumsum(0), (1, 0)).cpu().numpy()
                nbr[r] = (key % self.sch.nodes[a]).int().cpu().numpy()
        return indptr, nbr


class _Block:
    pass


class _MiniBatch:
    pass


def _minibatch(case, sch, seed, dev):
    """Layer-wise neighbour sampling: per hop one block, its destinations a prefix of its sources.  How many rows and
    edges there are belongs to the case; which vertices they are, and every list's order, comes from the seed."""
    g = _Graph(sch, 0, dev)
    T = sch.num_types
    dst = [torch.zeros(0, dtype=torch.int64, device=dev) for _ in range(T)]
    dst[sch.target] = g.targets(case["targets"])
    local = [torch.full((n,), -1, dtype=torch.int64, device=dev) for n in sch.nodes]
    blocks = []
    for fanout in (int(f) for f in case["fanout"].split(",")):
        src = list(dst)
        for t in range(T):
            local[t][src[t]] = torch.arange(src[t].numel(), device=dev)
        es, ed, et = [], [], []
        for r in range(sch.num_rels):
            s, d = sch.rel_src[r], sch.rel_dst[r]
            if dst[d].numel() == 0:
                continue
            row, u = g.neighbours(r, dst[d], fanout)
            new = torch.unique(u[local[s][u] < 0])
            if new.numel():
                new = new[torch.randperm(new.numel(), generator=g.gen, device=dev)]
                local[s][new] = src[s].numel() + torch.arange(new.numel(), device=dev)
                src[s] = torch.cat([src[s], new])
            es.append(local[s][u])
            ed.append(row)
            et.append(torch.full((row.numel(),), r, dtype=torch.int64, device=dev))
        for t in range(T):
            local[t][src[t]] = -1
        b = _Block()
        b.n_src, b.n_dst = [x.numel() for x in src], [x.numel() for x in dst]
        b.coo = torch.cat(es), torch.cat(ed), torch.cat(et)
        blocks.append(b)
        dst = src
    # the seed's vertices, and its order of the rows that each hop added
    gen = torch.Generator(dev).manual_seed(seed * 7919 + 12345)

    def order(n):
        return torch.randperm(n, generator=gen, device=dev)
    ids, moved = [], []
    for t in range(T):
        cuts = [0, blocks[0].n_dst[t]] + [b.n_src[t] for b in blocks]
        moved.append(torch.cat([lo + order(hi - lo) for lo, hi in zip(cuts, cuts[1:])]))
        x = torch.empty_like(dst[t])
        x[moved[t]] = order(sch.nodes[t])[dst[t]]
        ids.append(x.cpu().numpy())
    start = np.cumsum([0] + [m.numel() for m in moved])
    moved = torch.cat(moved)
    first_src, first_dst = (torch.tensor([int(start[t]) for t in ts], device=dev) for ts in (sch.rel_src, sch.rel_dst))
    for b in blocks:
        es, ed, et = b.coo
        del b.coo
        mix = order(es.numel())
        es, ed = moved[first_src[et] + es][mix], moved[first_dst[et] + ed][mix]
        b.edge_index = torch.stack([es, ed]).cpu().numpy()
        b.edge_type = et[mix].int().cpu().numpy()
    mb = _MiniBatch()
    mb.blocks, mb.ids, mb.labels, mb.grad_out = blocks[::-1], ids, None, None
    return mb


# ---- the model --------------------------------------------------------------------------------------------------
class _LayerWeights:
    w_rel = w_root = w_type = a_src = a_dst = ()
    w_sem = b_sem = q_sem = None


def _layers(case, sch, rng):
    def glorot(*shape, fans=None):
        a = math.sqrt(6.0 / sum(fans or shape))
        return rng.uniform(-a, a, size=shape).astype(np.float32)
    widths = [case["hidden"]] * (len(case["fanout"].split(",")) - 1) + [case["out"]]
    layers, dim = [], list(sch.feat)
    for i, H in enumerate(widths):
        lw = _LayerWeights()
        lw.in_dim, lw.out_dim, lw.relu = list(dim), H, i + 1 < len(widths)
        if case["layer"] == "mean":
            lw.w_rel = [glorot(dim[s], H) for s in sch.rel_src]
            lw.w_root = [glorot(dim[t], H) for t in range(sch.num_types)]
        else:
            k, D = case["heads"], H // case["heads"]
            lw.w_type = [glorot(dim[t], H) for t in range(sch.num_types)]
            lw.a_src = [glorot(k, D, fans=(D, 1)) for _ in sch.rels]
            lw.a_dst = [glorot(k, D, fans=(D, 1)) for _ in sch.rels]
            lw.w_sem, lw.q_sem = glorot(H, 128), glorot(128, fans=(128, 1))
            lw.b_sem = rng.uniform(-0.1, 0.1, 128).astype(np.float32)
        lw.bias = [rng.uniform(-0.1, 0.1, H).astype(np.float32) for _ in range(sch.num_types)]
        layers.append(lw)
        dim = [H] * sch.num_types
    return layers


def _like(old, flat, at):
    """The tensors of `old` (a list or one tensor) as consecutive views of `flat` from element at[0] on, same values."""
    if old is None or torch.is_tensor(old):
        if old is None:
            return None
        v = flat[at[0]: at[0] + old.numel()].view(old.shape)
        at[0] += old.numel()
        return v.copy_(old)
    return [_like(t, flat, at) for t in old]


GRADS = ("dw_rel", "dw_root", "dw_type", "da_src", "da_dst", "dw_sem", "db_sem", "dq_sem", "dbias")


def _flatten(model, first_layer_input_grad):
    """All weight gradients as views of one buffer, the way a program with one optimiser call or one gradient clip
    keeps them; returns the buffer."""
    def items(w):
        d = {**w, **w.get("dattn", {})}
        return [(k, d[k]) for k in GRADS if d.get(k) is not None]

    def tensors(x):
        return [x] if torch.is_tensor(x) else [t for t in x if t is not None]
    total = sum(t.numel() for w in model.weights for _, x in items(w) for t in tensors(x))
    flat, at = torch.zeros(total, device=model.dev, dtype=torch.float32), [0]
    for l, w in enumerate(model.weights):
        g = {k: _like(x, flat, at) for k, x in items(w)}
        old = model.layers[l]
        if model.attention:
            dattn = {k: v for k, v in g.items() if k != "dbias"}
            w.update(dattn=dattn, dbias=g["dbias"])
            model.layers[l] = binding.Layer(model.ctx, old.in_dim, old.out_dim, old.relu, None, None, w["bias"], None, None,
                                            g["dbias"], attn=w["attn"], dattn=dattn)
        else:
            w.update(g)
            model.layers[l] = binding.Layer(model.ctx, old.in_dim, old.out_dim, old.relu, w["w_rel"], w["w_root"], w["bias"],
                                            g["dw_rel"], g["dw_root"], g["dbias"],
                                            input_grad=first_layer_input_grad if l == 0 else None)
    return flat


class _State:
    pass


def prepare(case, seed):
    dev = torch.device("cuda", 0)
    sch = _Schema(case["family"])
    mode, attention = case["mode"], case["layer"] == "attention"
    learn = None if attention else sch.learnable
    s = _State()
    s.case, s.sch = case, sch
    feats = torch.Generator(dev).manual_seed(seed * 104729 + 7)
    stores = []
    for t, (n, f) in enumerate(zip(sch.nodes, sch.feat)):
        x = torch.randn((n, f), generator=feats, device=dev)
        if sch.learnable and sch.learnable[t]:
            x *= 0.1
        stores.append(x.cpu().numpy())
    classify = case["family"] == "academic" and not attention and mode in ("step", "train", "lists")
    s.model = Model(sch, sch.feat, stores, _layers(case, sch, np.random.default_rng([seed, 3])), dtype=case["dtype"],
                    loss="xent" if classify else "dot", target_type=sch.target, first_layer_input_grad=learn)
    del stores
    s.grads = _flatten(s.model, learn)
    s.pending = []
    if mode == "sampled":
        g = _Graph(sch, seed, dev)
        indptr, nbr = g.all_edges()
        s.sampler = s.model.ctx.hgnn_sampler_create(sch.nodes, indptr, nbr, np.cumsum([0] + [len(x) for x in nbr]))
        s.targets, s.seed = g.targets(case["targets"]).cpu().numpy(), seed
        s.fanouts = [int(f) for f in case["fanout"].split(",")]
        return s
    s.mb = _minibatch(case, sch, seed, dev)
    last = s.mb.blocks[-1]
    if classify:
        s.mb.labels = np.random.default_rng([seed, 4]).integers(0, case["out"], case["targets"])
    elif mode != "forward":
        s.mb.grad_out = [np.random.default_rng([seed, 5, t]).standard_normal((n, case["out"]), dtype=np.float32)
                         for t, n in enumerate(last.n_dst)]
    if mode == "lists":
        # edges by their ids in the whole graph, whose table of relations is registered once
        off = np.cumsum([0] + [sch.pairs[r[2]][2] for r in sch.rels])
        s.model.ctx.hgnn_set_edge_types(np.repeat(np.arange(sch.num_rels, dtype=np.int32), np.diff(off)))
        for i, b in enumerate(s.mb.blocks):
            u = np.random.default_rng([seed, 6, i]).random(len(b.edge_type))
            b.edge_id = off[b.edge_type] + (u * np.diff(off)[b.edge_type]).astype(np.int64)
        return s
    s.batch = s.model.prepare(s.mb)
    s.batch.graph.wait()
    if mode == "train":
        _optimizer(s)
    return s


def _optimizer(s):
    """Adam's state: fp32 masters and moments of all weights in one buffer each, and of the learnable tables."""
    model = s.model
    params = [p for w in model.weights for k in ("w_rel", "w_root", "bias") for p in w[k] if p is not None]
    grads = [p for w in model.weights for k in ("dw_rel", "dw_root", "dbias") for p in w[k] if p is not None]
    n = sum(p.numel() for p in params)
    s.master, s.m, s.v = (torch.zeros(n, device=model.dev) for _ in range(3))
    at = [0]
    masters = _like([p.float() for p in params], s.master, at)
    zeros = [torch.zeros_like(p, dtype=torch.float32) for p in params]
    s.list = model.ctx.AdamList(params, None if model.dtype == "f32" else masters, grads, _like(zeros, s.m, [0]), _like(zeros, s.v, [0]))
    s.params, s.step, s.tables = params, 0, {}
    for t in range(s.sch.num_types):
        if s.sch.learnable[t]:
            st = model.stores[t]
            s.tables[t] = [None if model.dtype == "f32" else st.float()] + [torch.zeros(st.shape, device=model.dev) for _ in range(2)]


def _input_grads(s, dx, n_rows):
    """The input gradients that the backward pass writes: those of the learnable types."""
    if s.sch.learnable is None or s.case["layer"] == "attention":
        return [dx]
    off = np.cumsum([0] + [n * f for n, f in zip(n_rows, s.sch.feat)])
    return [dx[off[t]: off[t + 1]] for t in range(s.sch.num_types) if s.sch.learnable[t]]


def run(s):
    model, mode = s.model, s.case["mode"]
    if mode == "forward":
        return {"h": model.run(s.batch, backward=False)["h"][-1]}
    if mode == "sampled":
        b = model.prepare_sampled(s.sampler, s.targets, s.fanouts, s.seed)
        out = model.run(b, backward=False)
        _keep(s, b)
        return {"h": out["h"][-1]}
    b = model.prepare(s.mb, use_edge_id=True) if mode == "lists" else s.batch
    out = model.run(b)
    res = {"h": out["h"][-1], "grads": s.grads, "dx": _input_grads(s, out["dx"][0], b.n_rows)}
    if model.loss == "xent":
        res["loss"] = out["loss"]
    if mode == "lists":
        _keep(s, b)
    if mode == "train":
        s.step += 1
        hp = (1e-3, 0.9, 0.999, 1e-8, s.step)
        model.ctx.hgnn_adam_update(s.list, *hp)
        for t, rows in zip(s.tables, res["dx"]):
            model.ctx.hgnn_adam_update_rows(model.stores[t], *s.tables[t], b.ids_dev[t], rows, *hp)
        res.update(master=s.master if model.dtype == "bf16" else s.params, m=s.m, v=s.v,
                   tables=[[model.stores[t]] + s.tables[t] for t in s.tables])
    return res


def _keep(s, batch):
    """A mini-batch's index arrays go back to the pool once the device work that reads them has finished."""
    done = torch.cuda.Event()
    done.record()
    s.pending.append((done, batch))
    while len(s.pending) > 2:
        e, b = s.pending.pop(0)
        e.synchronize()
        b.graph.release()


# ---- what a pass cannot do without ------------------------------------------------------------------------------
def work(case):
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    sch = _Schema(case["family"])
    mb = _minibatch(case, sch, 1, dev)
    es, backward = (2 if case["dtype"] == "bf16" else 4), case["mode"] not in ("forward", "sampled")
    attention = case["layer"] == "attention"
    widths = [case["hidden"]] * (len(mb.blocks) - 1) + [case["out"]]
    learn = sch.learnable if sch.learnable and not attention else [1] * sch.num_types
    dim, flops, weights = list(sch.feat), 0.0, 0
    # inputs read once (feature rows and their ids, index arrays), outputs written once
    nbytes = sum(n * (f * es + 8) for n, f in zip(mb.blocks[0].n_src, sch.feat))
    for l, (b, H) in enumerate(zip(mb.blocks, widths)):
        E = np.bincount(b.edge_type, minlength=sch.num_rels)
        rows = sum(b.n_dst[d] for d in sch.rel_dst)
        nbytes += 4 * (E.sum() + rows)
        if case["mode"] in ("lists", "sampled"):
            nbytes += 8 * E.sum() * (3 if case["mode"] == "lists" else 1)
        if backward:
            nbytes += 4 * (E.sum() + sum(b.n_src))
        want = learn if l == 0 else [1] * sch.num_types
        if attention:
            proj = sum(2.0 * n * f * H for n, f in zip(b.n_src, dim))
            agg = 4.0 * E.sum() * H + 2.0 * rows * H
            sem = 2.0 * rows * H * (128 + 1)
            flops += proj + agg + sem
            if backward:
                flops += 2 * proj + 2.5 * agg + 2 * sem
            weights += sum(f * H for f in dim) + 2 * sch.num_rels * H + H * 128 + 256 + sch.num_types * H
        else:
            for r in range(sch.num_rels):
                s, d = sch.rel_src[r], sch.rel_dst[r]
                weights += dim[s] * H
                if E[r]:
                    f = 2.0 * b.n_dst[d] * dim[s] * H
                    flops += f + E[r] * dim[s]
                    if backward:
                        flops += f + (f + E[r] * dim[s] if want[s] else 0)
            for t in range(sch.num_types):
                weights += dim[t] * H + H
                f = 2.0 * b.n_dst[t] * dim[t] * H
                flops += f + ((f + f * want[t]) if backward else 0)
        dim = [H] * sch.num_types
    nbytes += weights * es + sum(mb.blocks[-1].n_dst) * widths[-1] * es
    if backward:
        nbytes += weights * 4 + sum(n * f * es * w for n, f, w in zip(mb.blocks[0].n_src, sch.feat, learn))
        nbytes += sum(mb.blocks[-1].n_dst) * widths[-1] * es if case["family"] != "academic" or attention else case["targets"] * 8
    if case["mode"] == "train":
        emb = sum(n * f * w for n, f, w in zip(mb.blocks[0].n_src, sch.feat, learn))
        state = 24 if case["dtype"] == "f32" else 26          # moments and master read and written, parameter written
        nbytes += state * (weights + emb)
        flops += 12.0 * (weights + emb)
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    """bf16 storage: the rounding of what lies between the layers.  fp32: sums of a few thousand terms; where a hidden
    layer has a ReLU and gradients are taken, a unit whose pre-activation is within an fp32 rounding of zero may take
    the other decision, which moves a whole term of a gradient: of some 1e6 units a few do, so the gradients move by
    up to the root of that share."""
    if case["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 0.5}
    if case["mode"] in ("forward", "sampled") or case["fanout"].count(",") == 0:
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 2e-3, "max": 0.5}
