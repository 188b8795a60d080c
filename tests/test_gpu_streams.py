"""Streams and threads around the runner: what is complete when, and for whom."""
import threading

import numpy as np
import pytest

from tests.parity import prepare_inputs

pytestmark = pytest.mark.gpu


def _model(index=0, **kw):
    from paper_2408_08490_amd.runner import Model
    cfg, g, mb, ws = prepare_inputs(index, **kw)
    return Model(g.schema, g.feat_dim, g.stores, ws, dtype=cfg.dtype, loss=cfg.loss, target_type=mb.target_type), g, mb


def _busy(torch, ms=30):
    """Keeps the current stream occupied for some `ms` milliseconds."""
    a = torch.ones(4096, 4096, device="cuda")
    for _ in range(max(1, ms // 2)):
        a = a @ a * 1e-4
    return a


def test_id_lists_are_complete_for_every_stream_when_prepare_returns():
    """The caller's stream has work queued that outlasts the call; another stream reads the lists at once, as direct calls
    of the merge or the row update on that stream do."""
    import torch
    model, g, mb = _model(2, scale=0.05, batch=64)       # classified: the incoming gradient is the loss's
    _busy(torch, 4)
    torch.cuda.synchronize()
    for t in range(len(mb.ids)):               # what the allocator hands out next is not by chance the right answer
        torch.full((65536,), -1, device="cuda", dtype=torch.int64)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    keep = _busy(torch)
    bt = model.prepare(mb, g.edge_type, use_edge_id=True)
    with torch.cuda.stream(side):
        got, labels = [x.clone() for x in bt.ids_dev], bt.labels_dev.clone()
    side.synchronize()
    assert np.array_equal(labels.cpu().numpy(), mb.labels)
    for a, b in zip(got, mb.ids):
        assert np.array_equal(a.cpu().numpy(), b)
    torch.cuda.synchronize()
    del keep
    bt.graph.release()
    model.close()


def test_threads_that_prepare_at_once_get_their_own_lists():
    """Eight loader threads through one model's upload path: every list on the device is the caller's."""
    import torch
    model, g, mb = _model()
    wrong = []

    def loader(n):
        rng = np.random.default_rng(n)
        try:
            for i in range(200):
                lists = [rng.integers(0, 1 << 40, int(rng.integers(1, 3000))) for _ in range(3)]
                dev = model._uploads.put(lists)
                torch.cuda.synchronize()
                wrong.extend((n, i, k) for k, (a, b) in enumerate(zip(dev, lists)) if not np.array_equal(a.cpu().numpy(), b))
        except Exception as e:
            wrong.append((n, repr(e)))
    threads = [threading.Thread(target=loader, args=(n,)) for n in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong[:5]
    model.close()


def test_one_graph_from_two_streams():
    """The layers of one mini-batch on two streams in turn, the first calls made while the upload may be under way: the same
    bits as on one stream, forward and input gradient."""
    import torch
    model, g, mb = _model(2, scale=0.05, batch=256)
    ref = None
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for i in range(4):
        bt = model.prepare(mb, g.edge_type, use_edge_id=True)
        s = streams[i % 2]
        s.wait_stream(streams[1 - i % 2])      # the model's buffers are shared
        with torch.cuda.stream(s):
            out = model.run(bt, backward=False)
            got = [h.clone() for h in out["h"]]
        t = streams[1 - i % 2]
        t.wait_stream(s)
        with torch.cuda.stream(t):
            again = [h.clone() for h in model.run(bt, backward=False)["h"]]
        torch.cuda.synchronize()
        ref = ref or got
        assert all(torch.equal(a, b) for a, b in zip(ref, got)) and all(torch.equal(a, b) for a, b in zip(ref, again))
        bt.graph.release()
    model.close()


def test_the_first_call_on_a_graph_may_be_captured():
    """Nothing is known yet of the upload when the layer is captured (it is asked for inside the capture); the captured layer gives
    the eager bits on every replay."""
    import torch
    model, g, mb = _model(2, scale=0.05, batch=64)
    first = model.prepare(mb, g.edge_type, use_edge_id=True)
    out = model.run(first, backward=False)
    want, x0 = out["h"][0].clone(), out["x0"].clone()
    first.graph.release()
    bt = model.prepare(mb, g.edge_type, use_edge_id=True)
    sb, cb = model.ctx.hgnn_layer_workspace_bytes(bt.graph, 0, model.layers[0])
    bt.graph.host_view(0)                      # the build is over; the upload is not asked for
    torch.cuda.synchronize()
    sv, sc = (torch.empty(max(n, 256), device=model.dev, dtype=torch.uint8) for n in (sb, cb))
    h = torch.empty_like(want)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        model.ctx.hgnn_layer_fwd(bt.graph, 0, model.layers[0], x0, h, sv, sc)
    for _ in range(3):
        h.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(h, want)
    bt.graph.release()
    model.close()
