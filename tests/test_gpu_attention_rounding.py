"""The attention layer's backward against 64 bits where its one pass over a row's edges could cancel: a neighbour far from the
others with next to no weight, first or last in its row (the order of a row is an accident of the list)."""
from types import SimpleNamespace as NS

import numpy as np
import pytest

from oracle import hgnn_oracle as O
from tests.parity import rel_errors

pytestmark = pytest.mark.gpu

N, F, H, HEADS, DEG = 192, 64, 64, 2, 9


def _case(scale, first):
    """N destinations with DEG ordinary neighbours and one of their own whose features are `scale` times as long and whose
    score is -60 (-12 behind the LeakyReLU)."""
    rng = np.random.default_rng(17)
    x = rng.standard_normal((3 * N, F))
    a_src, a_dst = (rng.standard_normal((HEADS, F // HEADS)) * 0.3 for _ in range(2))
    far = rng.standard_normal((N, HEADS, F // HEADS)) * scale
    far += ((-60.0 - (far * a_src).sum(2)) / (a_src * a_src).sum(1))[:, :, None] * a_src
    x[2 * N:] = far.reshape(N, F)
    src = rng.integers(0, 2 * N, (N, DEG))
    own = 2 * N + np.arange(N)[:, None]
    src = np.concatenate([own, src] if first else [src, own], axis=1)
    f32 = lambda a: np.ascontiguousarray(a, dtype=np.float32)
    lw = NS(in_dim=[F], out_dim=H, relu=False, w_rel=(), w_root=(), w_type=[np.eye(F, H, dtype=np.float32)], a_src=[f32(a_src)],
            a_dst=[f32(a_dst)], w_sem=f32(rng.standard_normal((H, 128)) / H), b_sem=f32(rng.standard_normal(128) * 0.1),
            q_sem=f32(rng.standard_normal(128) * 0.1), bias=[f32(rng.standard_normal(H))])
    block = NS(n_src=[3 * N], n_dst=[N], edge_index=np.stack([src.reshape(-1), np.repeat(np.arange(N), DEG + 1)]),
               edge_type=np.zeros(N * (DEG + 1), np.int32))
    mb = NS(ids=[np.arange(3 * N)], blocks=[block], labels=None, grad_out=[f32(rng.standard_normal((N, H)))])
    return NS(num_types=1, num_rels=1, rel_src=[0], rel_dst=[0]), f32(x), lw, mb


@pytest.mark.parametrize("scale", [1.0, 30.0, 1000.0])
@pytest.mark.parametrize("first", [True, False])
def test_attention_gradients_with_a_far_neighbour_of_next_to_no_weight(scale, first):
    """Tolerance: what the softmax brings.  __expf is exp2 of a rounded product, so a weight is off by 2^-24 times its
    exponent (up to 12 here, plus the score's own rounding: 32 products and sums of magnitude up to 60), up to
    4e-6 of the gradients (2e-7 measured; 3e-6 at 1000 times the length).  Taken relative to the first neighbour, the one
    pass lost 2.5e-5 of da_dst at 30 times the length and 8e-4 at 1000 times."""
    import torch
    from paper_2408_08490_amd.runner import Model
    sch, x, lw, mb = _case(scale, first)
    model = Model(sch, [F], [x], [lw], dtype="f32", loss="dot", target_type=0)
    bt = model.prepare(mb)
    out = model.run(bt)
    torch.cuda.synchronize()
    b = mb.blocks[0]
    edges = [(b.edge_index[0], b.edge_index[1])]
    h, cache = O.rgat_layer_forward([x], edges, [0], [0], b.n_dst, lw.w_type, lw.a_src, lw.a_dst, lw.w_sem, lw.b_sem, lw.q_sem, lw.bias,
                                    False, HEADS)
    ref = O.rgat_layer_backward(cache, mb.grad_out)
    d = model.weights[0]["dattn"]
    got = dict(h=out["h"][0], da_src=d["da_src"][0], da_dst=d["da_dst"][0], dw_type=d["dw_type"][0], dx=out["dx"][0])
    want = dict(h=h[0], da_src=ref["da_src"][0], da_dst=ref["da_dst"][0], dw_type=ref["dw_type"][0], dx=ref["dx"][0])
    errors = {k: rel_errors(got[k].float().cpu().numpy().ravel(), np.asarray(want[k]).ravel())[1] for k in got}
    assert all(e < 1e-5 for e in errors.values()), errors
    bt.graph.release()
    model.close()
