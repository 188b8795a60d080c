"""The bf16 forward of a layer with a ReLU on 64x64 tiles, whose K-steps take the aggregate's value and remainder together: segments
that end inside a K-step, an odd and an even number of steps, a destination type without a root term, relations without edges, rows
and columns that end inside a tile."""
from types import SimpleNamespace as NS

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _bf16(a):
    import torch
    return torch.from_numpy(np.float32(a)).bfloat16().double().numpy()


@pytest.mark.parametrize("widths,root", [((8, 8), True), ((64, 64), False), ((72, 56), True), ((136, 264), True), ((192, 64), False)])
def test_forward_with_both_planes_in_one_step(widths, root):
    import torch
    from paper_2408_08490_amd.runner import Model
    rng = np.random.default_rng(sum(widths))
    n_src, n_dst, H = 900, 2100, 264   # 165 tiles of 64x64: more than the split reduction takes, fewer large ones than it takes for those
    draw = lambda *s: _bf16(rng.standard_normal(s))
    x = [draw(n, f) for n, f in zip((n_src, n_dst), widths)]
    rels = [(0, 1), (1, 1), (0, 1)]   # the last one without edges
    edges = [(rng.integers(0, (n_src, n_dst)[s], 5000), rng.integers(0, n_dst, 5000)) for s, _ in rels[:2]]
    w_rel = [draw(widths[s], H) for s, _ in rels]
    w_root = [None, draw(widths[1], H) if root else None]
    bias = [draw(H) for _ in range(2)]
    lw = NS(in_dim=list(widths), out_dim=H, relu=True, w_type=[], w_rel=w_rel, w_root=w_root, bias=bias)
    block = NS(n_src=[n_src, n_dst], n_dst=[0, n_dst], edge_index=np.concatenate([np.stack(e) for e in edges], 1),
               edge_type=np.repeat(np.arange(2, dtype=np.int32), 5000))
    model = Model(NS(num_types=2, num_rels=3, rel_src=[s for s, _ in rels], rel_dst=[d for _, d in rels]), list(widths), x, [lw], dtype="bf16",
                  loss="dot", target_type=1)
    bt = model.prepare(NS(ids=[np.arange(n_src), np.arange(n_dst)], blocks=[block], labels=None, grad_out=None))
    got = model.run(bt, backward=False)["h"][0].double().cpu().numpy().reshape(n_dst, H)
    bt.graph.release()
    model.close()
    # in 64 bits, with the sum of the magnitudes of each unit's terms
    pre, size = np.tile(bias[1], (n_dst, 1)), np.tile(np.abs(bias[1]), (n_dst, 1))
    for (src, dst), (s, _), w in zip(edges, rels, w_rel):
        deg = np.maximum(np.bincount(dst, minlength=n_dst), 1)[:, None]
        for total, f in ((pre, lambda a: a), (size, np.abs)):
            z = np.zeros((n_dst, widths[s]))
            np.add.at(z, dst, f(x[s])[src])
            total += z / deg @ f(w)
    if root:
        pre += x[1] @ w_root[1]
        size += np.abs(x[1]) @ np.abs(w_root[1])
    # the aggregate keeps 2^-17 of itself as value and remainder, the sums are fp32, the output is rounded to bf16 once
    assert (np.abs(got - np.maximum(pre, 0)) <= 2.0 ** -8 * np.abs(pre) + 2.0 ** -16 * size).all()
