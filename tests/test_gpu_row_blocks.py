"""Kernels that walk blocks of rows: the attention aggregation, whose block keeps the indices of its rows in LDS (1024 of them)
and sums a head over 1 to 64 lanes, and the backward products around the lines between tiles of 64 and of 128 rows."""
from types import SimpleNamespace as NS

import numpy as np
import pytest

from oracle import hgnn_oracle as O
from tests.parity import rel_errors
from workloads.synth import bf16_round

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 1e-2}   # fp32 sums; terms and results rounded to 2^-9


def _run(dtype, n_src, n_dst, src, dst, width, H, heads=0, root=True, input_grad=True):
    """Forward and backward of a layer of one relation (attention with heads > 0): pairs (this library, 64 bits)."""
    import torch
    from paper_2408_08490_amd.runner import Model
    rng = np.random.default_rng(len(src) + H)
    rnd = (lambda a: bf16_round(np.float32(a))) if dtype == "bf16" else np.float32
    x = [rnd(rng.standard_normal((n, width))) for n in (n_src, n_dst)]
    lw = NS(in_dim=[width, width], out_dim=H, relu=False, w_type=[], w_rel=[], w_root=[], bias=[rnd(rng.standard_normal(H)) for _ in range(2)])
    weight = lambda: rnd(rng.standard_normal((width, H)) / width ** 0.5)
    if heads:
        lw.w_type = [weight(), weight()]
        lw.a_src, lw.a_dst = ([rnd(rng.standard_normal((heads, H // heads)) * 0.3)] for _ in range(2))
        lw.w_sem, lw.b_sem, lw.q_sem = (rnd(rng.standard_normal(s) * 0.1) for s in ((H, 128), 128, 128))
    else:
        lw.w_rel, lw.w_root = [weight()], [None, weight() if root else None]
    block = NS(n_src=[n_src, n_dst], n_dst=[0, n_dst], edge_index=np.stack([src, dst]), edge_type=np.zeros(len(src), np.int32))
    grad = [np.zeros((0, H), np.float32), rnd(rng.standard_normal((n_dst, H)))]
    mb = NS(ids=[np.arange(n_src), np.arange(n_dst)], blocks=[block], labels=None, grad_out=grad)
    model = Model(NS(num_types=2, num_rels=1, rel_src=[0], rel_dst=[1]), [width, width], x, [lw], dtype=dtype, loss="dot", target_type=1)
    bt = model.prepare(mb)
    out = model.run(bt, need_input_grad=input_grad)
    torch.cuda.synchronize()
    if heads:
        want, cache = O.rgat_layer_forward(x, [(src, dst)], [0], [1], block.n_dst, lw.w_type, lw.a_src, lw.a_dst, lw.w_sem, lw.b_sem,
                                           lw.q_sem, lw.bias, False, heads)
        g = O.rgat_layer_backward(cache, grad)
        dx, pairs = g["dx"], list(zip(model.weights[0]["dattn"]["dw_type"], g["dw_type"]))
    else:
        want, cache = O.rgcn_layer_forward(x, [(src, dst)], [0], [1], block.n_dst, lw.w_rel, lw.w_root, lw.bias, False)
        dx, dw_rel, dw_root, _ = O.rgcn_layer_backward(cache, grad)
        pairs = [(model.weights[0]["dw_rel"][0], dw_rel[0])] + ([(model.weights[0]["dw_root"][1], dw_root[1])] if root else [])
    pairs += [(out["h"][0], want[1])]
    if input_grad:
        pairs += [(out["dx"][0], np.concatenate([np.ravel(d) for d in dx]))]
    errors = [rel_errors(got.float().cpu().numpy().ravel(), np.ravel(ref))[1] for got, ref in pairs]
    bt.graph.release()
    model.close()
    return errors


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("H,heads", [(8, 2), (16, 2), (16, 1), (64, 2), (64, 1), (128, 1), (256, 1)])
def test_attention_rows_beyond_the_staged_indices(H, heads, dtype):
    rng = np.random.default_rng(H)
    degrees = [0, 1, 4, 5, 1019, 3, 2, 8, 0, 1100] + [int(k) for k in rng.integers(0, 9, 290)]
    n_src, n_dst = 1200, len(degrees)
    src = np.concatenate([rng.permutation(n_src)[:k] for k in degrees])
    dst = np.repeat(np.arange(n_dst), degrees)
    order = rng.permutation(len(src))
    errors = _run(dtype, n_src, n_dst, src[order], dst[order], 64, H, heads)
    assert max(errors) < TOL[dtype], errors


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_dst", [6000, 12289, 16100, 20500])
def test_backward_tiles(n_dst, dtype):
    """Two products of 256 columns per destination row: about 200, 420, 540 and 690 tiles of 128 in bf16, 380, 700, 840 and 970
    in fp32, whose weight gradients are cut finer (in 64x64 ones but for fp32's 380)."""
    n_src = 60
    src = np.concatenate([np.arange(n_dst) % n_src, (np.arange(0, n_dst, 3) * 7 + 1) % n_src])
    dst = np.concatenate([np.arange(n_dst), np.arange(0, n_dst, 3)])
    errors = _run(dtype, n_src, n_dst, src, dst, 256, 96)
    assert max(errors) < TOL[dtype], errors


def _tiles(dtype, n, F, H, segments, both=True):
    """Tiles of 128 of the two backward products of a layer of `segments` segments (relations and root terms) over n rows: blocks of
    rows for the input gradients (where `both` are computed), slices of the reduction for the weight gradients (a 1/640 of all K-steps
    each)."""
    bk, least = (64, 32) if dtype == "bf16" else (32, 4)
    up = lambda a, b: -(-a // b)
    cols, cols_h = segments * up(F, 128), up(H, 128)
    da = cols * up(n, 128) if both else 0
    steps = up(cols * cols_h * up(n, bk) + da * up(H, bk), 640)
    return da + cols * cols_h * up(n, bk * min(64, max(least, steps)))


def tiles_and_columns(case):
    """Rows (a ragged last tile), tiles of 128 and the columns in blocks of 128 and of 64 with the number of types, of a case below."""
    dtype, F, H, segments, tiles, _ = case[:6]
    n = next(n for n in range(64, 400000, 8) if _tiles(dtype, n, F, H, segments, len(case) == 6) >= tiles) + 3
    return n, _tiles(dtype, n, F, H, segments, len(case) == 6), (segments * -(-F // 128), segments * -(-F // 64), 1)


# dtype, width of the input, of the output, segments, tiles of 128 (or a few more), the edge of the tiles it takes.  Both sides of every
# line of bwd_small_tiles: 256 where the line for the width lies below it; in bf16 1000, 880, 680, 500 and 460 for outputs of up to 64,
# 128, 256, 352 and more; in fp32 1600 where much of a large tile is padding, none for outputs of up to 64, for 160 from 256 to 512 (but not
# with one column block per block of rows) and then 1350, for up to 192 1000, 320 800, and 700 beyond.
TILE_CASES = [("f32", 256, 96, 2, 244, 64), ("f32", 256, 96, 2, 256, 128), ("f32", 256, 96, 2, 500, 128), ("f32", 256, 96, 2, 512, 64),
              ("f32", 256, 96, 2, 1336, 64), ("f32", 256, 96, 2, 1350, 128), ("f32", 128, 96, 1, 300, 64), ("f32", 128, 64, 2, 1610, 64),
              ("f32", 192, 96, 2, 1585, 64), ("f32", 192, 96, 2, 1600, 128), ("f32", 192, 352, 2, 710, 64),
              ("f32", 256, 176, 2, 985, 64), ("f32", 256, 176, 2, 1000, 128), ("f32", 256, 264, 2, 785, 64), ("f32", 256, 264, 2, 800, 128),
              ("f32", 128, 352, 2, 685, 64), ("f32", 128, 352, 2, 700, 128), ("bf16", 256, 64, 2, 985, 64), ("bf16", 256, 64, 2, 1000, 128),
              ("bf16", 256, 96, 2, 865, 64), ("bf16", 256, 96, 2, 880, 128), ("bf16", 256, 200, 2, 665, 64), ("bf16", 256, 200, 2, 680, 128),
              ("bf16", 128, 264, 2, 485, 64), ("bf16", 128, 264, 2, 500, 128), ("bf16", 128, 400, 2, 445, 64), ("bf16", 128, 400, 2, 460, 128)]
# without the input gradients (a seventh entry): bf16 320; fp32 700, everywhere for outputs of up to 64, 1600 for 129 to 192
TILE_CASES += [("bf16", 512, 400, 2, 270, 64, "dw"), ("bf16", 512, 400, 2, 320, 128, "dw"), ("f32", 512, 500, 2, 400, 64, "dw"), ("f32", 512, 500, 2, 704, 128, "dw"),
               ("f32", 512, 176, 2, 704, 64, "dw"), ("f32", 512, 64, 2, 320, 64, "dw")]
# and between the lines
TILE_CASES += [("f32", 256, 96, 2, tiles, edge) for tiles, edge in ((372, 128), (388, 128), (508, 64), (520, 64), (760, 64), (772, 64))]
TILE_CASES += [("f32", 64, 96, 2, 300, 64), ("f32", 64, 96, 2, 400, 64), ("f32", 192, 96, 2, 300, 64), ("f32", 128, 352, 2, 300, 64),
               ("f32", 128, 352, 2, 400, 64), ("f32", 128, 352, 2, 690, 64), ("f32", 128, 352, 2, 704, 128)]
TILE_CASES += [("bf16", 256, 96, 2, tiles, 64) for tiles in (244, 300, 504, 516)] + [("bf16", 128, 264, 2, tiles, 64) for tiles in (240, 300)]


@pytest.mark.parametrize("case", TILE_CASES, ids=lambda c: "-".join(map(str, c)))
def test_backward_tiles_on_both_sides_of_the_lines(case):
    dtype, F, H, segments, tiles, _ = case[:6]
    n_src, (n_dst, have, _) = 60, tiles_and_columns(case)
    assert tiles <= have <= tiles + 32
    src = np.concatenate([np.arange(n_dst) % n_src, (np.arange(0, n_dst, 3) * 7 + 1) % n_src])
    dst = np.concatenate([np.arange(n_dst), np.arange(0, n_dst, 3)])
    errors = _run(dtype, n_src, n_dst, src, dst, F, H, root=segments == 2, input_grad=len(case) == 6)
    assert max(errors) < TOL[dtype], errors


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_attention_with_several_rows_per_lane_group(dtype):
    """33000 merged rows of 256 floats: lane groups walk two rows each in the forward, four in the backward by rows and four in
    the one over the transpose (69000 source rows), beside 40 source rows of 17 to 300 entries."""
    rng = np.random.default_rng(41)
    n_src, n_dst = 36_000, 33_000
    src, dst = rng.integers(40, n_src, n_dst), rng.permutation(n_dst)
    lengths = np.linspace(17, 300, 40).astype(int)
    src = np.concatenate([src, np.repeat(np.arange(40), lengths)])
    dst = np.concatenate([dst, *(rng.permutation(n_dst - 5)[:k] for k in lengths)])   # five rows keep one edge; some have several
    order = rng.permutation(len(src))
    errors = _run(dtype, n_src, n_dst, src[order], dst[order], 32, 256, 8)
    assert max(errors) < TOL[dtype], errors
