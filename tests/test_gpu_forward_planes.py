"""The bf16 forward of a layer with a ReLU on 64x64 tiles, which multiplies the aggregate's value and then its remainder with the
same weights: segments that end inside a K-step, an odd and an even number of steps, a destination type without a root term,
relations without edges, rows and columns that end inside a tile.  And the order of a row's sums, which is that of 128x128 tiles."""
from types import SimpleNamespace as NS

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _bf16(a):
    import torch
    return torch.from_numpy(np.float32(a)).bfloat16().double().numpy()


@pytest.mark.parametrize("widths,root", [((8, 8), True), ((64, 64), False), ((72, 56), True), ((136, 264), True), ((192, 64), False)])
def test_forward_with_value_and_remainder(widths, root):
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


@pytest.mark.parametrize("dtype,relu,H,blocks", [("bf16", True, 264, 106), ("bf16", False, 264, 106), ("f32", True, 264, 139), ("f32", False, 264, 106)])
def test_a_row_has_the_same_bits_on_small_and_large_tiles(dtype, relu, H, blocks):
    """The first `blocks` blocks of 128 rows alone, which 64x64 tiles multiply, and with one more block behind them, which takes the
    launch over the line to 128x128 ones: every sum is formed in the same order, so that the rows' outputs are the same bits."""
    import torch
    from paper_2408_08490_amd.runner import Model
    rng = np.random.default_rng(blocks)
    F, n_src, most = 136, 500, (blocks + 1) * 128
    x = np.float32(rng.standard_normal((most, F)))
    w = [np.float32(rng.standard_normal((F, H)) / F ** 0.5) for _ in range(3)]
    lw = NS(in_dim=[F], out_dim=H, relu=relu, w_type=[], w_rel=w[:2], w_root=w[2:], bias=[np.float32(rng.standard_normal(H))])
    ends = [(rng.integers(0, n_src, 2 * most), rng.permutation(2 * most) % most) for _ in range(2)]
    got = []
    for rows in (blocks * 128, most):
        edges = [np.stack([s[d < rows], d[d < rows]]) for s, d in ends]
        block = NS(n_src=[rows], n_dst=[rows], edge_index=np.concatenate(edges, 1),
                   edge_type=np.repeat(np.arange(2, dtype=np.int32), [e.shape[1] for e in edges]))
        model = Model(NS(num_types=1, num_rels=2, rel_src=[0, 0], rel_dst=[0, 0]), [F], [x[:rows]], [lw], dtype=dtype, loss="dot", target_type=0)
        bt = model.prepare(NS(ids=[np.arange(rows)], blocks=[block], labels=None, grad_out=None))
        got.append(model.run(bt, backward=False)["h"][0].clone().view(rows, H)[:blocks * 128])
        torch.cuda.synchronize()
        bt.graph.release()
        model.close()
    assert torch.equal(*got)
