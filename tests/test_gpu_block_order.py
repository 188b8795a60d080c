"""Launches whose blocks change places with the launch's size: the forward aggregation with the weight transposes in front of
its rows (up to 2048 blocks) and behind them, and the attention fusion with one and with four rows per lane group."""
from types import SimpleNamespace as NS

import numpy as np
import pytest

from oracle import hgnn_oracle as O
from tests.parity import rel_errors
from workloads.synth import bf16_round

pytestmark = pytest.mark.gpu


def _run(dtype, kind, n_dst, widths, H, heads=1):
    """Output of a layer of one relation, every destination row with one or two of 50 sources, beside 64 bits."""
    import torch
    from paper_2408_08490_amd.runner import Model
    rng = np.random.default_rng(n_dst)
    rnd = (lambda a: bf16_round(np.float32(a))) if dtype == "bf16" else np.float32
    n_src = 50
    src = np.concatenate([np.arange(n_dst) % n_src, (np.arange(0, n_dst, 3) * 7 + 1) % n_src])
    dst = np.concatenate([np.arange(n_dst), np.arange(0, n_dst, 3)])
    x = [rnd(rng.standard_normal((n, f))) for n, f in zip((n_src, n_dst), widths)]
    lw = NS(in_dim=list(widths), out_dim=H, relu=False, w_type=[], w_rel=[], w_root=[], bias=[rnd(rng.standard_normal(H)) for _ in range(2)])
    if kind == "attention":
        lw.w_type = [rnd(rng.standard_normal((f, H)) / f ** 0.5) for f in widths]
        lw.a_src, lw.a_dst = ([rnd(rng.standard_normal((heads, H // heads)) * 0.3)] for _ in range(2))
        lw.w_sem, lw.b_sem, lw.q_sem = (rnd(rng.standard_normal(s) * 0.1) for s in ((H, 128), 128, 128))
    else:
        lw.w_rel = [rnd(rng.standard_normal((widths[0], H)) / widths[0] ** 0.5)]
        lw.w_root = [None, rnd(rng.standard_normal((widths[1], H)) / widths[1] ** 0.5)]
    block = NS(n_src=[n_src, n_dst], n_dst=[0, n_dst], edge_index=np.stack([src, dst]), edge_type=np.zeros(len(src), np.int32))
    mb = NS(ids=[np.arange(n_src), np.arange(n_dst)], blocks=[block], labels=None, grad_out=[np.zeros((0, H), np.float32), x[1][:, :1] * np.ones(H, np.float32)])
    model = Model(NS(num_types=2, num_rels=1, rel_src=[0], rel_dst=[1]), list(widths), x, [lw], dtype=dtype, loss="dot", target_type=1)
    bt = model.prepare(mb)
    got = model.run(bt, backward=False)["h"][0].float().cpu().numpy().reshape(-1, H)
    torch.cuda.synchronize()
    if kind == "attention":
        want, _ = O.rgat_layer_forward(x, [(src, dst)], [0], [1], [0, n_dst], lw.w_type, lw.a_src, lw.a_dst, lw.w_sem, lw.b_sem, lw.q_sem,
                                       lw.bias, False, heads)
    else:
        want, _ = O.rgcn_layer_forward(x, [(src, dst)], [0], [1], [0, n_dst], lw.w_rel, lw.w_root, lw.bias, False)
    bt.graph.release()
    model.close()
    return rel_errors(got[-n_dst:].ravel(), np.asarray(want[1]).ravel())[1]


# rows of 1 KB take four to a block: one row more or less than the 2048 blocks there are with the transposes
@pytest.mark.parametrize("dtype,F,ragged", [("bf16", 512, False), ("f32", 256, False), ("bf16", 512, True), ("f32", 256, True)])
@pytest.mark.parametrize("more", [-4, 0, 1, 5])
def test_transposes_in_front_of_the_rows_and_behind(dtype, F, ragged, more):
    root = F // 2 if ragged else F
    n_dst = (2048 - (F + root) // 32) * 4 + more
    assert _run(dtype, "mean", n_dst, (F, root), 32) < (1e-5 if dtype == "f32" else 1e-2)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_dst,H", [(16383, 256), (16384, 256), (16399, 256), (32771, 128)])
def test_fusion_rows_per_lane_group(dtype, n_dst, H):
    assert _run(dtype, "attention", n_dst, (64, 64), H, heads=4) < (1e-5 if dtype == "f32" else 1e-2)
