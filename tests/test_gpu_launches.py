"""What the layer calls enqueue: their kernels counted in a captured graph, against hgnn_layer_launch_count; and the
per-relation launch structure against the merged one where both form the same sums."""
import ctypes

import numpy as np
import pytest

from tests.parity import prepare_inputs

pytestmark = pytest.mark.gpu


def _kernel_nodes(torch, graph):
    hip = ctypes.CDLL("libamdhip64.so")
    g, n = ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(g, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(g, nodes, ctypes.byref(n)) == 0
    kinds = []
    for x in nodes:
        t = ctypes.c_int(-1)
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(x), ctypes.byref(t)) == 0
        kinds.append(t.value)
    return sum(t == 0 for t in kinds)   # hipGraphNodeTypeKernel


@pytest.mark.parametrize("index,scale,batch", [(0, 1.0, None), (5, 1.0, None), (2, 0.05, 64), (1, 0.05, 256), (2, 0.05, 2048)])
def test_forward_launches_counted_in_a_captured_graph(index, scale, batch):
    """Small batches and many relations (the split reduction adds its partial tiles up in a kernel of its own), and launches
    that need none.  Replayed three times between eager passes, the graph gives the eager bits."""
    import torch
    from paper_2408_08490_amd.runner import Model
    cfg, g, mb, ws = prepare_inputs(index, scale=scale, batch=batch)
    model = Model(g.schema, g.feat_dim, g.stores, ws, dtype=cfg.dtype, loss=cfg.loss, target_type=mb.target_type)
    bt = model.prepare(mb, g.edge_type, use_edge_id=True)
    bt.graph.wait()
    want = [h.clone() for h in model.run(bt, backward=False)["h"][:len(model.layers)]]
    torch.cuda.synchronize()
    graphs, outs = [], []
    x = model.run(bt, backward=False)
    torch.cuda.synchronize()
    for l, lp in enumerate(model.layers):       # one graph per layer
        xin = x["x0"] if l == 0 else x["h"][l - 1]
        sb, cb = model.ctx.hgnn_layer_workspace_bytes(bt.graph, l, lp)
        sv, sc = (torch.empty(max(n, 256), device=model.dev, dtype=torch.uint8) for n in (sb, cb))
        h = torch.empty_like(want[l])
        cg = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(cg):
            model.ctx.hgnn_layer_fwd(bt.graph, l, lp, xin, h, sv, sc)
        counted, said = _kernel_nodes(torch, cg), model.ctx.hgnn_layer_launch_count(bt.graph, l, lp)[0]
        graphs.append((cg, h, sv, sc, counted, said))
    for _ in range(3):
        for l, (cg, h, *_rest) in enumerate(graphs):
            h.fill_(7.0)
            cg.replay()
            torch.cuda.synchronize()
            assert torch.equal(h, want[l]), l
            model.run(bt, backward=False)
            torch.cuda.synchronize()
    assert [c for *_x, c, s in graphs] == [s for *_x, c, s in graphs]
    bt.graph.release()
    model.close()


def test_per_relation_launches_form_the_merged_sums_before_a_relu():
    """One relation, no root term: both launch structures take one product over the same terms in the same order, so an fp32
    layer with a ReLU gives the same bits (a sum formed on other units decides units near zero differently).  1024 rows of
    256: the merged launch is beyond the split reduction."""
    import torch
    from types import SimpleNamespace as NS
    from paper_2408_08490_amd.runner import Model
    n, F, H = 1024, 192, 256
    rng = np.random.default_rng(8)
    sch = NS(num_types=1, num_rels=1, rel_src=[0], rel_dst=[0])
    lw = NS(in_dim=[F], out_dim=H, relu=True, w_rel=[rng.standard_normal((F, H)).astype(np.float32)], w_root=[None],
            bias=[rng.standard_normal(H).astype(np.float32)], w_type=[])
    model = Model(sch, [F], [rng.standard_normal((2000, F)).astype(np.float32)], [lw], dtype="f32", loss="dot", target_type=0)
    E = 8 * n
    block = NS(n_src=[1500], n_dst=[n], edge_index=np.stack([rng.integers(0, 1500, E), rng.integers(0, n, E)]),
               edge_type=np.zeros(E, np.int32))
    mb = NS(ids=[rng.permutation(2000)[:1500]], blocks=[block], labels=None, grad_out=None)
    bt = model.prepare(mb)
    merged = model.run(bt, backward=False)["h"][0].clone()
    naive = model.run(bt, backward=False, naive=True)["h"][0].clone()
    torch.cuda.synchronize()
    assert torch.equal(merged, naive)
    bt.graph.release()
    model.close()
