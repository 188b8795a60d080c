"""Source vertices with many destinations: rows of the transpose around the length at which a block takes them, and around one
and several pieces, over two relations, in all three transposed sums (one width, ragged widths, attention)."""
from types import SimpleNamespace as NS

import numpy as np
import pytest

from oracle import hgnn_oracle as O
from tests.parity import rel_errors
from workloads.synth import bf16_round

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 16, 17, 18, 127, 128, 129, 255, 256, 257, 700, 1500, 3, 0]   # entries of the first sources; then one each


def _case(kind, dtype, widths, H, heads):
    rng = np.random.default_rng(29)
    n_src, n_dst = 90, 800
    rnd = (lambda a: bf16_round(np.float32(a))) if dtype == "bf16" else np.float32
    lengths = LENGTHS + [1] * (n_src - len(LENGTHS))
    src = np.repeat(np.arange(n_src), lengths)
    dst = np.concatenate([rng.permutation(2 * n_dst)[:k] for k in lengths])   # place 0 .. n_dst - 1: relation 0
    rel, dst = (dst // n_dst).astype(np.int32), dst % n_dst
    order = rng.permutation(len(src))
    src, dst, rel = src[order], dst[order], rel[order]
    block = NS(n_src=[n_src, n_dst], n_dst=[0, n_dst], edge_index=np.stack([src, dst]), edge_type=rel)
    edges = [(src[rel == r], dst[rel == r]) for r in range(2)]
    x = [rnd(rng.standard_normal((n, f))) for n, f in zip((n_src, n_dst), widths)]
    lw = NS(in_dim=list(widths), out_dim=H, relu=False, w_type=[], w_rel=[], w_root=[], bias=[rnd(rng.standard_normal(H)) for _ in range(2)])
    if kind == "attention":
        lw.w_type = [rnd(rng.standard_normal((f, H)) / f ** 0.5) for f in widths]
        lw.a_src, lw.a_dst = ([rnd(rng.standard_normal((heads, H // heads)) * 0.3) for _ in range(2)] for _ in range(2))
        lw.w_sem, lw.b_sem, lw.q_sem = (rnd(rng.standard_normal(s) * 0.1) for s in ((H, 128), 128, 128))
    else:
        lw.w_rel = [rnd(rng.standard_normal((widths[0], H)) / widths[0] ** 0.5) for _ in range(2)]
        lw.w_root = [None, rnd(rng.standard_normal((widths[1], H)) / widths[1] ** 0.5)]
    grad = [np.zeros((0, H), np.float32), rnd(rng.standard_normal((n_dst, H)))]
    mb = NS(ids=[np.arange(n_src), np.arange(n_dst)], blocks=[block], labels=None, grad_out=grad)
    return NS(num_types=2, num_rels=2, rel_src=[0, 0], rel_dst=[1, 1]), x, lw, mb, edges


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("kind,widths,H,heads", [("mean", (8, 8), 16, 1), ("mean", (128, 128), 32, 1), ("mean", (520, 520), 32, 1),
                                                 ("mean", (1032, 1032), 16, 1), ("mean", (40, 72), 32, 1), ("mean", (24, 136), 16, 1),
                                                 ("attention", (64, 64), 8, 1), ("attention", (64, 32), 64, 2), ("attention", (128, 128), 256, 8)])
def test_long_transpose_rows(kind, widths, H, heads, dtype):
    """Input gradients against 64 bits: sums of up to 1500 fp32 terms (1e-6 of their norm and less), in bf16 over terms
    and results rounded to 2^-9.  Three runs of the mean layer give the same bits: the pieces are added
    in a fixed order (the attention layer's relation scores are added with atomics)."""
    import torch
    from paper_2408_08490_amd.runner import Model
    sch, x, lw, mb, edges = _case(kind, dtype, widths, H, heads)
    model = Model(sch, list(widths), x, [lw], dtype=dtype, loss="dot", target_type=1)
    bt = model.prepare(mb)
    runs = []
    for _ in range(3):
        runs.append(model.run(bt)["dx"][0].clone())
    torch.cuda.synchronize()
    if kind == "mean":
        assert torch.equal(runs[0], runs[1]) and torch.equal(runs[0], runs[2])
    if kind == "attention":
        _, cache = O.rgat_layer_forward(x, edges, [0, 0], [1, 1], mb.blocks[0].n_dst, lw.w_type, lw.a_src, lw.a_dst, lw.w_sem, lw.b_sem,
                                        lw.q_sem, lw.bias, False, heads)
        want = O.rgat_layer_backward(cache, mb.grad_out)["dx"]
    else:
        _, cache = O.rgcn_layer_forward(x, edges, [0, 0], [1, 1], mb.blocks[0].n_dst, lw.w_rel, lw.w_root, lw.bias, False)
        want = O.rgcn_layer_backward(cache, mb.grad_out)[0]
    got = runs[0].float().cpu().numpy()
    cut = x[0].size
    tol = 1e-5 if dtype == "f32" else 1e-2
    errors = [rel_errors(g.ravel(), np.asarray(w).ravel())[1] for g, w in ((got[:cut], want[0]), (got[cut:], want[1]))]
    assert all(e < tol for e in errors), errors
    bt.graph.release()
    model.close()


MIXES = {"few": LENGTHS + [1] * 60, "many": [17, 18, 31, 64, 65, 127, 128, 129, 300, 2] * 360}   # the second: 4320 pieces


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("mix", ["few", "many"])
@pytest.mark.parametrize("kind,widths,H,heads", [("mean", (8, 8), 16, 1), ("mean", (64, 64), 32, 1), ("mean", (128, 128), 32, 1), ("mean", (264, 264), 16, 1),
                                                 ("mean", (40, 32), 32, 1), ("mean", (24, 136), 16, 1), ("attention", (64, 32), 64, 2),
                                                 ("attention", (32, 64), 16, 1), ("attention", (64, 64), 128, 4)])
def test_long_rows_that_are_destinations(kind, widths, H, heads, mix, dtype):
    """Long rows of both types, most of them destinations as well, whose own term the piece that finishes a row adds once; few
    and more pieces than the chip holds blocks.  Another gradient runs over the same work areas in between, so that partial sums
    left from the run before would show; the mean layer runs one launch per type too, each over all pieces with one type's
    wanted.  Bounds as above."""
    import torch
    from paper_2408_08490_amd.runner import Model
    rng = np.random.default_rng(31)
    rnd = (lambda a: bf16_round(np.float32(a))) if dtype == "bf16" else np.float32
    lengths = MIXES[mix]
    n_dst, n_src = [len(lengths) - 7, 800], [len(lengths), 805]
    if mix == "few":
        n_dst[0] = 70
    places = n_dst[1] + n_dst[0]   # of relation 0 (0 -> 1), then of relation 1 (0 -> 0)
    src = np.repeat(np.arange(n_src[0]), [min(k, places) for k in lengths])
    at = np.concatenate([rng.permutation(places)[:k] for k in lengths])
    back = (rng.integers(0, 40, 3000), rng.integers(0, n_dst[0], 3000))   # relation 2 (1 -> 0): 40 sources of some 75 entries
    src, dst, rel = (np.concatenate(z) for z in ((src, back[0]), (np.where(at < n_dst[1], at, at - n_dst[1]), back[1]),
                                                 ((at >= n_dst[1]).astype(np.int32), np.full(3000, 2, np.int32))))
    order = rng.permutation(len(src))
    src, dst, rel = src[order], dst[order], rel[order]
    rel_src, rel_dst = [0, 0, 1], [1, 0, 0]
    edges = [(src[rel == r], dst[rel == r]) for r in range(3)]
    x = [rnd(rng.standard_normal((n, f))) for n, f in zip(n_src, widths)]
    lw = NS(in_dim=list(widths), out_dim=H, relu=False, w_type=[], w_rel=[], w_root=[], bias=[rnd(rng.standard_normal(H)) for _ in range(2)])
    if kind == "attention":
        lw.w_type = [rnd(rng.standard_normal((f, H)) / f ** 0.5) for f in widths]
        lw.a_src, lw.a_dst = ([rnd(rng.standard_normal((heads, H // heads)) * 0.3) for _ in range(3)] for _ in range(2))
        lw.w_sem, lw.b_sem, lw.q_sem = (rnd(rng.standard_normal(s) * 0.1) for s in ((H, 128), 128, 128))
        _, cache = O.rgat_layer_forward(x, edges, rel_src, rel_dst, n_dst, lw.w_type, lw.a_src, lw.a_dst, lw.w_sem, lw.b_sem, lw.q_sem, lw.bias, False, heads)
        want = lambda grad: O.rgat_layer_backward(cache, grad)["dx"]
    else:
        lw.w_rel = [rnd(rng.standard_normal((widths[s], H)) / widths[s] ** 0.5) for s in rel_src]
        lw.w_root = [rnd(rng.standard_normal((f, H)) / f ** 0.5) for f in widths]
        _, cache = O.rgcn_layer_forward(x, edges, rel_src, rel_dst, n_dst, lw.w_rel, lw.w_root, lw.bias, False)
        want = lambda grad: O.rgcn_layer_backward(cache, grad)[0]
    grads = [[rnd(rng.standard_normal((n, H)) * s) for n in n_dst] for s in (1, 8)]
    block = NS(n_src=n_src, n_dst=n_dst, edge_index=np.stack([src, dst]), edge_type=rel)
    mb = NS(ids=[np.arange(n) for n in n_src], blocks=[block], labels=None, grad_out=grads[0])
    model = Model(NS(num_types=2, num_rels=3, rel_src=rel_src, rel_dst=rel_dst), list(widths), x, [lw], dtype=dtype, loss="dot", target_type=1)
    bt = model.prepare(mb)
    given = [torch.from_numpy(np.concatenate([g.ravel() for g in gs])).to(bt.grad_out_dev) for gs in grads]
    got = []
    for which, naive in ((0, False), (1, False), (0, False)) + (((1, True),) if kind == "mean" else ()):
        bt.grad_out_dev = given[which]
        got.append((which, model.run(bt, naive=naive)["dx"][0].clone()))
    torch.cuda.synchronize()
    if kind == "mean":
        assert torch.equal(got[0][1], got[2][1])
    cut, refs = x[0].size, [want(gs) for gs in grads]
    for which, dx in got:
        dx = dx.float().cpu().numpy()
        errors = [rel_errors(g.ravel(), np.asarray(w).ravel())[1] for g, w in ((dx[:cut], refs[which][0]), (dx[cut:], refs[which][1]))]
        assert all(e < (1e-5 if dtype == "f32" else 1e-2) for e in errors), (which, errors)
    bt.graph.release()
    model.close()
