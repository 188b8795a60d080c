"""The forward products on both sides of the lines between tiles of 64 and of 128 rows and columns (fwd_small_tiles), with rows,
columns and a K-segment that end inside a tile."""
from types import SimpleNamespace as NS

import numpy as np
import pytest

from workloads.synth import bf16_round

pytestmark = pytest.mark.gpu

# dtype, ReLU, columns, tiles of 128x128, the edge of the tiles it takes: 320; in fp32 with a ReLU 420, and 64 again between 512 and
# 2000; up to 64 columns 1000 in bf16, everywhere in fp32
CASES = [("bf16", True, 264, 318, 64), ("bf16", True, 264, 321, 128), ("bf16", False, 264, 318, 64), ("bf16", False, 264, 321, 128),
         ("f32", False, 264, 318, 64), ("f32", False, 264, 321, 128), ("f32", True, 264, 417, 64), ("f32", True, 264, 420, 128),
         ("f32", True, 264, 510, 128), ("f32", True, 264, 513, 64), ("f32", True, 264, 1998, 64), ("f32", True, 264, 2001, 128),
         ("bf16", True, 50, 999, 64), ("bf16", True, 50, 1000, 128), ("bf16", False, 64, 1000, 128), ("f32", True, 50, 1010, 64),
         ("f32", False, 64, 1010, 64)]


@pytest.mark.parametrize("dtype,relu,H,tiles,edge", CASES)
def test_forward_on_both_sides_of_the_lines(dtype, relu, H, tiles, edge):
    """Bounds: an fp32 sum of at most 81 terms of either sign is off by 81 * 2^-24 of the sum of the magnitudes at most; in bf16 the
    output is rounded once, to 2^-9, and without a ReLU, whose layers keep the remainder, the aggregate too."""
    import torch
    from paper_2408_08490_amd.runner import Model
    rng = np.random.default_rng(tiles)
    F, n_src = 40, 700
    rows = tiles // -(-H // 128) * 128 - 61
    rnd = (lambda a: bf16_round(np.float32(a))) if dtype == "bf16" else np.float32
    x = [rnd(rng.standard_normal((n, F))) for n in (n_src, rows)]
    w = [rnd(rng.standard_normal((F, H)) / F ** 0.5) for _ in range(2)]
    bias = rnd(rng.standard_normal(H))
    dst = np.concatenate([np.arange(rows), np.arange(0, rows, 2), np.arange(0, rows, 2)])
    src = rng.integers(0, n_src, len(dst))
    lw = NS(in_dim=[F, F], out_dim=H, relu=relu, w_type=[], w_rel=[w[0]], w_root=[None, w[1]], bias=[None, bias])
    block = NS(n_src=[n_src, rows], n_dst=[0, rows], edge_index=np.stack([src, dst]), edge_type=np.zeros(len(dst), np.int32))
    model = Model(NS(num_types=2, num_rels=1, rel_src=[0], rel_dst=[1]), [F, F], x, [lw], dtype=dtype, loss="dot", target_type=1)
    bt = model.prepare(NS(ids=[np.arange(n_src), np.arange(rows)], blocks=[block], labels=None, grad_out=None))
    got = model.run(bt, backward=False)["h"][0].view(rows, H).double().cpu()
    bt.graph.release()
    model.close()
    s, d = torch.from_numpy(src), torch.from_numpy(dst)
    deg = torch.bincount(d, minlength=rows).clamp_(min=1).double()[:, None]

    def terms(f):
        z = torch.zeros((rows, F), dtype=torch.float64).index_add_(0, d, f(torch.from_numpy(x[0]).double())[s]) / deg
        a, b = (f(torch.from_numpy(m).double()) for m in w)
        return z @ a, f(torch.from_numpy(x[1]).double()) @ b + f(torch.from_numpy(bias).double())
    pre, size = sum(terms(lambda a: a)), terms(torch.abs)
    bound = 2.0 ** -17 * sum(size)
    if dtype == "bf16":
        bound += 2.0 ** -8 * pre.abs() + (2.0 ** -8 * size[0] if not relu else 2.0 ** -16 * size[0])
    assert bool(((got - (pre.clamp(min=0) if relu else pre)).abs() <= bound).all())
