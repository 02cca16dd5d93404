"""The radius search of an event alone (its planes shared by several workgroups)
and inside a batch large enough for one workgroup per plane: the same edges, in
every form of the search, for dense and sparse embeddings of both padded widths."""
import numpy as np
import pytest

from paper_2508_07423_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _edges(etx, w, weights, batch, options):
    b = etx.to_device(batch)
    p = etx.Pipeline(w, weights)
    for key, value in options.items():
        etx.etx_set_option(p.ctx, getattr(etx, "ETX_OPT_" + key), value)
    p.run(b)
    res = p.results(b)
    p.close()
    return res


@pytest.mark.parametrize("fast,split,sort_min", [(0, 0, 512), (0, 1, 1024), (1, 0, 128), (1, 1, 128), (1, 1, 0)])
@pytest.mark.parametrize("name,trained,tracks,events", [("c1", False, 50, 60), ("c1", True, 50, 60),
                                                        ("c2", True, 200, 24), ("c2", False, 40, 24),
                                                        ("c3", False, 600, 24)])
def test_parts_give_the_same_graph(name, trained, tracks, events, fast, split, sort_min):
    from paper_2508_07423_amd import etx
    w = synth.WORKLOADS[name].with_(gnn_steps=1)
    weights = synth.trained_weights(synth.WORKLOADS[name]) if trained else synth.xavier_weights(w)
    batch = synth.generate_batch(w.with_(tracks=("fixed", tracks)), events, first=7)
    options = dict(RADIUS_FAST=fast, RADIUS_SPLIT=split, RADIUS_SORT_MIN=sort_min)
    whole = _edges(etx, w, weights, batch, options)
    plain = _edges(etx, w, weights, batch, dict(RADIUS_SINGLE_PASS=0))      # the two-pass form, no fast path
    assert np.array_equal(whole["src"], plain["src"]) and np.array_equal(whole["dst"], plain["dst"])
    ho, eo = batch["hit_off"], whole["edge_off"]
    for i in (0, events - 1):
        ev = dict(synth.event_slice(batch, i), hit_off=np.array([0, ho[i + 1] - ho[i]], np.int64))
        one = _edges(etx, w, weights, ev, options)
        part = slice(eo[i], eo[i + 1])
        assert np.array_equal(one["src"] + ho[i], whole["src"][part])
        assert np.array_equal(one["dst"] + ho[i], whole["dst"][part])
