"""The attention layer's fusion backward, which takes a block's rows against up to four relations of their type at a time: as many
relations as one to three such turns hold, rows that end inside a turn of four, a type's mask and bias with and without a ReLU."""
from types import SimpleNamespace as NS

import numpy as np
import pytest

from oracle import hgnn_oracle as O

pytestmark = pytest.mark.gpu

F, H, HEADS = 32, 64, 2


@pytest.mark.parametrize("rels", [1, 2, 3, 4, 5, 6, 8, 11])
@pytest.mark.parametrize("rows,relu", [(1, False), (63, True), (66, False), (129, True)])
def test_relations_of_a_type_in_turns(rels, rows, relu):
    """Tolerance: each sum's terms are fp32 products rounded a few times, at most 2^-18 of the magnitudes summed; the semantic gradients
    subtract the relations' weighted mean from each of them, which costs up to a factor of 16 here."""
    import torch
    from paper_2408_08490_amd.runner import Model
    rng = np.random.default_rng(rels)
    n_src = rows + 40
    x = np.float32(rng.standard_normal((n_src, F)))
    w = lambda *s: np.float32(rng.standard_normal(s) * 0.3)
    lw = NS(in_dim=[F], out_dim=H, relu=relu, w_rel=(), w_root=(), w_type=[w(F, H)], a_src=[w(HEADS, H // HEADS) for _ in range(rels)],
            a_dst=[w(HEADS, H // HEADS) for _ in range(rels)], w_sem=w(H, 128), b_sem=w(128), q_sem=w(128), bias=[w(H)])
    edges = [(rng.integers(0, n_src, 3 * rows), rng.integers(0, rows, 3 * rows)) for _ in range(rels)]
    block = NS(n_src=[n_src], n_dst=[rows], edge_index=np.concatenate([np.stack(e) for e in edges], 1),
               edge_type=np.repeat(np.arange(rels, dtype=np.int32), 3 * rows))
    g = np.float32(rng.standard_normal((rows, H)))
    model = Model(NS(num_types=1, num_rels=rels, rel_src=[0] * rels, rel_dst=[0] * rels), [F], [x], [lw], dtype="f32", loss="dot", target_type=0)
    bt = model.prepare(NS(ids=[np.arange(n_src)], blocks=[block], labels=None, grad_out=[g]))
    model.run(bt)
    torch.cuda.synchronize()
    f64 = lambda a: np.asarray(a, np.float64)
    _, cache = O.rgat_layer_forward([f64(x)], edges, [0] * rels, [0] * rels, [rows], lw.w_type, lw.a_src, lw.a_dst, lw.w_sem, lw.b_sem, lw.q_sem,
                                    lw.bias, relu, HEADS)
    ref = O.rgat_layer_backward(cache, [f64(g)])
    d = model.weights[0]["dattn"]
    for name, got, want in [("dbias", model.weights[0]["dbias"][0], ref["dbias"][0]), ("dw_type", d["dw_type"][0], ref["dw_type"][0])] + [
            (k, d[k], ref[k]) for k in ("dw_sem", "db_sem", "dq_sem")]:
        got, want = got.double().cpu().numpy().ravel(), np.asarray(want).ravel()
        assert np.linalg.norm(got - want) <= 6e-5 * np.linalg.norm(want) + 1e-6, name
    bt.graph.release()
    model.close()


@pytest.mark.parametrize("dtype,rels", [("f32", 5), ("bf16", 6)])
def test_several_rows_of_a_lane_group_against_two_turns_of_relations(dtype, rels):
    """32805 rows of 256 columns: a lane group takes its rows in two trips, of which some groups have only the first, and keeps its
    shares of four relations' dots, then of the others', from trip to trip; the semantic products run on tiles of 128 rows.  The ReLU's
    decisions are the ones the library took, so that a unit within a rounding of zero does not move a whole term.  Bounds as above; in
    bf16 the projected features' gradient is rounded to 2^-9 in front of dW_type's sums."""
    import torch
    from paper_2408_08490_amd.runner import Model
    from workloads.synth import bf16_round
    rng = np.random.default_rng(rels)
    rows, n_src, H = 32805, 33000, 256
    rnd = (lambda a: bf16_round(np.float32(a))) if dtype == "bf16" else np.float32
    draw = lambda *s: rnd(rng.standard_normal(s) * 0.3)
    x = rnd(rng.standard_normal((n_src, F)))
    lw = NS(in_dim=[F], out_dim=H, relu=True, w_rel=(), w_root=(), w_type=[draw(F, H)], a_src=[draw(HEADS, H // HEADS) for _ in range(rels)],
            a_dst=[draw(HEADS, H // HEADS) for _ in range(rels)], w_sem=draw(H, 128), b_sem=draw(128), q_sem=draw(128), bias=[draw(H)])
    edges = [(rng.integers(0, n_src, rows), rng.permutation(rows)) for _ in range(rels)]
    block = NS(n_src=[n_src], n_dst=[rows], edge_index=np.concatenate([np.stack(e) for e in edges], 1),
               edge_type=np.repeat(np.arange(rels, dtype=np.int32), rows))
    g = rnd(rng.standard_normal((rows, H)))
    model = Model(NS(num_types=1, num_rels=rels, rel_src=[0] * rels, rel_dst=[0] * rels), [F], [x], [lw], dtype=dtype, loss="dot", target_type=0)
    bt = model.prepare(NS(ids=[np.arange(n_src)], blocks=[block], labels=None, grad_out=[g]))
    h = model.run(bt)["h"][0].view(rows, H).float().cpu().numpy()
    torch.cuda.synchronize()
    f64 = lambda a: np.asarray(a, np.float64)
    want, cache = O.rgat_layer_forward([f64(x)], edges, [0] * rels, [0] * rels, [rows], [f64(w) for w in lw.w_type], [f64(a) for a in lw.a_src],
                                       [f64(a) for a in lw.a_dst], f64(lw.w_sem), f64(lw.b_sem), f64(lw.q_sem), [f64(lw.bias[0])], False, HEADS)
    assert np.linalg.norm(h - np.maximum(want[0], 0)) <= (1e-5 if dtype == "f32" else 2.0 ** -8) * np.linalg.norm(want[0])
    ref = O.rgat_layer_backward(cache, [f64(g) * (h > 0)])
    d = model.weights[0]["dattn"]
    for name, got, want in [("dbias", model.weights[0]["dbias"][0], ref["dbias"][0]), ("dw_type", d["dw_type"][0], ref["dw_type"][0])] + [
            (k, d[k], ref[k]) for k in ("dw_sem", "db_sem", "dq_sem")]:
        got, want = got.double().cpu().numpy().ravel(), np.asarray(want).ravel()
        tol = 1e-2 if dtype == "bf16" and name == "dw_type" else 6e-5
        assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want) + 1e-6, (name, np.linalg.norm(got - want) / np.linalg.norm(want))
    bt.graph.release()
    model.close()
