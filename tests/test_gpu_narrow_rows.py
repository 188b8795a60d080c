"""Input rows of 16 bytes, the narrowest there are: one piece per row, forward and backward, merged and straight from the
feature stores, with more rows per type than a wavefront owns and fewer."""
import pytest

from tests.parity import run_case

pytestmark = pytest.mark.gpu


def _narrow(width):
    def edit(cfg, g, mb, ws):
        g.stores = [s[:, :width].copy() for s in g.stores]
        g.feat_dim = [width] * len(g.stores)
        ws[0].in_dim = [width] * len(g.stores)
        ws[0].w_rel = [w[:width].copy() for w in ws[0].w_rel]
        ws[0].w_root = [None if w is None else w[:width].copy() for w in ws[0].w_root]
    return edit


@pytest.mark.parametrize("index,width,batch", [(1, 4, 129), (1, 4, 3), (2, 8, 129), (2, 8, 3)])
def test_rows_of_one_piece(index, width, batch):
    rep = run_case(index, scale=0.02, batch=batch, verbose=True, check_gather=True, check_two_step=True, check_naive=True,
                   cfg_edit=_narrow(width))
    bad = {k: v for k, v in rep.items() if v == "MISMATCH"}
    assert rep["ok"], {"bad": bad, "report": {k: v for k, v in rep.items() if isinstance(v, tuple)}}
