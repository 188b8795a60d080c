"""The forward product of small launches, whose K-steps are dealt to blocks and wavefronts: tiles that one block takes whole
and tiles that are split, whose partial sums a second kernel adds up; tiles of 16, 32 and 64 columns."""
from types import SimpleNamespace as NS

import numpy as np
import pytest

from oracle import hgnn_oracle as O
from tests.parity import rel_errors
from workloads.synth import bf16_round

pytestmark = pytest.mark.gpu


def _forward(dtype, widths, H, relu, kernels):
    import torch
    from paper_2408_08490_amd.runner import Model
    rng = np.random.default_rng(sum(widths))
    n_src, n_dst = 210, 130
    src, dst = rng.integers(0, n_src, 900), rng.integers(0, n_dst, 900)
    draw = lambda *s: np.float32(rng.standard_normal(s))
    rnd = bf16_round if dtype == "bf16" else np.float32
    x = [rnd(draw(n, f)) for n, f in zip((n_src, n_dst), widths)]
    lw = NS(in_dim=list(widths), out_dim=H, relu=relu, w_type=[], w_rel=[rnd(draw(widths[0], H) / widths[0] ** 0.5)],
            w_root=[None, rnd(draw(widths[1], H) / widths[1] ** 0.5)], bias=[rnd(draw(H)) for _ in range(2)])
    block = NS(n_src=[n_src, n_dst], n_dst=[0, n_dst], edge_index=np.stack([src, dst]), edge_type=np.zeros(900, np.int32))
    mb = NS(ids=[np.arange(n_src), np.arange(n_dst)], blocks=[block], labels=None, grad_out=None)
    model = Model(NS(num_types=2, num_rels=1, rel_src=[0], rel_dst=[1]), list(widths), x, [lw], dtype=dtype, loss="dot", target_type=1)
    bt = model.prepare(mb)
    runs = [model.run(bt, backward=False)["h"][0].clone() for _ in range(2)]
    torch.cuda.synchronize()
    assert torch.equal(*runs)
    assert model.ctx.hgnn_layer_launch_count(bt.graph, 0, model.layers[0])[0] == 1 + kernels   # and the aggregation
    want, _ = O.rgcn_layer_forward(x, [(src, dst)], [0], [1], block.n_dst, lw.w_rel, lw.w_root, lw.bias, relu)
    # sums of 2816 fp32 terms at most; in bf16 the output and, without a ReLU, the aggregate are rounded to 2^-9
    assert rel_errors(runs[0].float().cpu().numpy().ravel(), np.asarray(want[1]).ravel())[1] < (1e-5 if dtype == "f32" else 2.0 ** -8)
    bt.graph.release()
    model.close()


# K-steps of 32 of a tile of type 1 (relation and root term): 1 + 1 .. 4 + 4 (two for each of four wavefronts) in one kernel; 4 + 5
# and more are split, up to 80 steps of few blocks with a step for each wavefront and beyond with two (88: 11 pieces)
@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("widths,kernels", [((16, 32), 1), ((128, 128), 1), ((128, 132), 2), ((160, 128), 2), ((512, 256), 2), ((1536, 1280), 2)])
def test_forward_of_few_tiles(widths, kernels, relu):
    _forward("f32", widths, 70, relu, kernels)


# widths of the output on both sides of the tiles of 16 and 32 columns, and ones that are no multiple of four, whose rows are not aligned;
# in one kernel and split, the bf16 layer with a ReLU with its remainder's steps
@pytest.mark.parametrize("dtype,relu", [("f32", False), ("bf16", False), ("bf16", True)])
@pytest.mark.parametrize("H", [2, 5, 10, 16, 17, 22, 32, 33, 64])
@pytest.mark.parametrize("widths,kernels", [((64, 64), 1), ((1536, 1280), 2)])
def test_widths_of_the_output(widths, kernels, H, dtype, relu):
    _forward(dtype, widths, H, relu, kernels)
