"""fp32 products on the bf16 matrix cores (three planes per operand) where they could lose: values and sums beyond the planes'
range (those tiles are multiplied again on the fp32 MFMA), values near the lower end of fp32, and sums of very few terms.
A large value meets a small one, so that what comes out is finite and every row or column has a scale of its own to be
compared on."""
from types import SimpleNamespace as NS

import numpy as np
import pytest

from oracle import hgnn_oracle as O
from tests.parity import rel_errors

pytestmark = pytest.mark.gpu

f32 = lambda a: np.ascontiguousarray(a, dtype=np.float32)


def _mean_layer(n, F, H, edit=lambda x, w, g: None, seed=3):
    """One type, one relation, no activation: n destinations with one neighbour each.  Returns what the library and the oracle
    make of it: h, dw_rel, dw_root, dx."""
    import torch
    from paper_2408_08490_amd.runner import Model
    rng = np.random.default_rng(seed)
    x, g = f32(rng.standard_normal((n + 8, F))), f32(rng.standard_normal((n, H)))
    w = [f32(rng.standard_normal((F, H)) / np.sqrt(F)) for _ in range(2)]
    edit(x, w, g)
    src = rng.integers(0, n + 8, n)
    lw = NS(in_dim=[F], out_dim=H, relu=False, w_rel=[w[0]], w_root=[w[1]], bias=[None], w_type=[])
    block = NS(n_src=[n + 8], n_dst=[n], edge_index=np.stack([src, np.arange(n)]), edge_type=np.zeros(n, np.int32))
    model = Model(NS(num_types=1, num_rels=1, rel_src=[0], rel_dst=[0]), [F], [x], [lw], dtype="f32", loss="dot", target_type=0)
    bt = model.prepare(NS(ids=[np.arange(n + 8)], blocks=[block], labels=None, grad_out=[g]))
    out = model.run(bt)
    torch.cuda.synchronize()
    got = dict(h=out["h"][0].view(n, H), dw_rel=model.weights[0]["dw_rel"][0], dw_root=model.weights[0]["dw_root"][0],
               dx=out["dx"][0].view(n + 8, F))
    got = {k: v.cpu().numpy().astype(np.float64) for k, v in got.items()}
    bt.graph.release()
    model.close()
    h, cache = O.rgcn_layer_forward([x], [(src, np.arange(n))], [0], [0], [n], [w[0]], [w[1]], [None], False)
    dx, dw_rel, dw_root, _ = O.rgcn_layer_backward(cache, [g])
    return got, dict(h=h[0], dw_rel=dw_rel[0], dw_root=dw_root[0], dx=dx[0])


BIG = 2.0 ** 110      # beyond the planes, whose operands are scaled by 2^24


# forward: 64x64 tiles (more than the split reduction takes) and 128x128; backward: 64x64 and 128x128 tiles
@pytest.mark.parametrize("n,F,H", [(4200, 32, 512), (16600, 128, 512), (300, 64, 128)])
@pytest.mark.parametrize("large", ["feature", "gradient"])
def test_products_of_values_beyond_the_planes(n, F, H, large):
    """A feature column of 2^110 against a weight row of 2^-110 (forward and dW, a row of which is large), or a gradient column
    of 2^110 against a weight column of 2^-110 (dX and dW, a column of which is large)."""
    def edit(x, w, g):
        if large == "feature":
            x[:, 3] *= BIG
        else:
            g[:, 5] *= BIG
        for m in w:
            if large == "feature":
                m[3] /= BIG
            else:
                m[:, 5] /= BIG
    got, want = _mean_layer(n, F, H, edit)
    for r in (got, want):
        if large == "feature":
            r["dx"][:, 3] *= BIG
        else:
            r["h"][:, 5] *= BIG
        for k in ("dw_rel", "dw_root"):
            if large == "feature":
                r[k][3] /= BIG
            else:
                r[k][:, 5] /= BIG
    errors = {k: max(rel_errors(got[k], want[k])) for k in got}
    assert all(e < 1e-4 for e in errors.values()), errors     # the storage type's tolerance, as everywhere


def test_an_infinite_feature_reaches_its_own_outputs_only():
    """4200 rows of 32 against 512 columns, all weights positive: the rows that read the infinite feature are infinite (not
    NaN), the others as without it; backward, dW of that feature alone is not finite."""
    def positive(x, w, g):
        for m in w:
            np.abs(m, out=m)
            m += np.float32(0.01)
        x[:, 0] = np.abs(x[:, 0])

    def infinite(x, w, g):
        positive(x, w, g)
        x[17, 0] = np.inf
    before, _ = _mean_layer(4200, 32, 512, positive)
    with np.errstate(invalid="ignore"):
        after, want = _mean_layer(4200, 32, 512, infinite)
    assert np.array_equal(np.isinf(after["h"]), np.isinf(want["h"])) and np.isinf(after["h"]).any() and not np.isnan(after["h"]).any()
    same = np.isfinite(want["h"])
    assert np.allclose(after["h"][same], before["h"][same], rtol=1e-5, atol=1e-5)
    for k in ("dw_rel", "dw_root"):
        assert np.isfinite(after[k][1:]).all() and np.allclose(after[k][1:], before[k][1:], rtol=1e-4, atol=1e-3)
    assert not np.isfinite(after["dw_root"][0]).any()
    assert np.allclose(after["dx"], before["dx"], rtol=1e-4, atol=1e-4)


@pytest.mark.parametrize("scale", [1e-30, 1e-34, 1e-36])
def test_products_of_values_near_the_lower_end(scale):
    """Gradients and features of that size: every normal fp32 value has three normal planes (bound: 1e-6 of the norm, as at 1)."""
    for edit in (lambda x, w, g: np.multiply(g, np.float32(scale), out=g), lambda x, w, g: np.multiply(x, np.float32(scale), out=x)):
        got, want = _mean_layer(4200, 32, 512, edit)
        errors = {k: np.linalg.norm(got[k] - want[k]) / np.linalg.norm(want[k]) for k in got}
        assert all(e < 1e-6 for e in errors.values()), errors


@pytest.mark.parametrize("rows", [1, 2, 3, 4])
def test_weight_gradients_over_very_few_rows(rows):
    """One product is rounded once: at most 2^-24 of it.  Sums of a few terms: a rounding per term, measured on the sum of the
    magnitudes."""
    keep = {}

    def edit(x, w, g):
        keep.update(x=x.astype(np.float64), g=g.astype(np.float64))
    got, want = _mean_layer(rows, 64, 64, edit)
    magnitude = np.abs(keep["x"][:rows]).T @ np.abs(keep["g"])
    assert (np.abs(got["dw_root"] - want["dw_root"]) <= 1.01 * rows * 2.0 ** -24 * magnitude).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [200, 20000, 33000])
def test_attention_products_beyond_the_planes(dtype, n):
    """Two relations into one type.  Column 3 of the projected features is 2^110 times as large and meets a row of W_s that much
    smaller (projection in fp32, scores, dW_s with its column sums); column 5 is 2^-120 or 2^-116 times as large and meets a row that
    much larger (dm).  Tiles of 64 rows and, where there are 512 of 128 and more (33000 rows), of 128."""
    import torch
    from paper_2408_08490_amd.runner import Model
    from workloads import bf16_round
    F = H = 64
    # dW's column 5 sums 2n terms of 1 / DOWN and either sign, some 4 sqrt(2n) / DOWN: with 2^120 that is 2^130 for 33000 rows, beyond fp32
    UP, DOWN = 2.0 ** 110, 2.0 ** (-120 if n <= 20000 else -116)
    rng = np.random.default_rng(23)
    store = bf16_round if dtype == "bf16" else (lambda a: a)
    x, g = store(f32(rng.standard_normal((2 * n, F)))), f32(rng.standard_normal((n, H)))
    col = np.ones(H)
    col[3], col[5] = UP, DOWN
    g /= col.astype(np.float32)                                  # dm then is of order 1 / col
    g = store(f32(g))
    wt = store(f32(rng.standard_normal((F, H)) / 8 * col))
    a = [store(f32(rng.standard_normal((1, H)) * 0.3 / col)) for _ in range(4)]
    ws = store(f32(rng.standard_normal((H, 128)) / 8 / col[:, None]))
    lw = NS(in_dim=[F], out_dim=H, relu=False, w_rel=(), w_root=(), w_type=[wt], a_src=a[:2], a_dst=a[2:], w_sem=ws,
            b_sem=store(f32(rng.standard_normal(128) * 0.1)), q_sem=store(f32(rng.standard_normal(128) * 0.1)), bias=[None])
    E = 3 * n
    ei = [np.stack([rng.integers(0, 2 * n, E), rng.integers(0, n, E)]) for _ in range(2)]
    block = NS(n_src=[2 * n], n_dst=[n], edge_index=np.concatenate(ei, axis=1), edge_type=np.repeat(np.int32([0, 1]), E))
    model = Model(NS(num_types=1, num_rels=2, rel_src=[0, 0], rel_dst=[0, 0]), [F], [x], [lw], dtype=dtype, loss="dot", target_type=0)
    bt = model.prepare(NS(ids=[np.arange(2 * n)], blocks=[block], labels=None, grad_out=[g]))
    out = model.run(bt)
    torch.cuda.synchronize()
    h, cache = O.rgat_layer_forward([x], [tuple(e) for e in ei], [0, 0], [0, 0], [n], lw.w_type, lw.a_src, lw.a_dst, ws, lw.b_sem,
                                    lw.q_sem, [None], False, 1)
    ref = O.rgat_layer_backward(cache, [g])
    d = model.weights[0]["dattn"]
    pairs = dict(h=(out["h"][0], h[0], 1 / col), dw_type=(d["dw_type"][0], ref["dw_type"][0], col), dx=(out["dx"][0], ref["dx"][0], 1.0),
                 da_src=(d["da_src"][1], ref["da_src"][1], 1 / col), dw_sem=(d["dw_sem"], ref["dw_sem"], 1 / col[:, None]),
                 db_sem=(d["db_sem"], ref["db_sem"], 1.0), dq_sem=(d["dq_sem"], ref["dq_sem"], 1.0))
    errors = {}
    for k, (got, want, s) in pairs.items():
        want = np.asarray(want) * s
        errors[k] = rel_errors(got.double().cpu().numpy().reshape(want.shape) * s, want)[1]
    tol = 1e-4 if dtype == "f32" else 2e-2
    assert all(e < tol for e in errors.values()), errors
    bt.graph.release()
    model.close()
