"""An event alone (node update with one workgroup per 16 nodes or with workgroups
of four waves, edge workgroups without a tile leave at once) and inside a batch large enough for the full workgroups: the same
edges, scores and labels, bit for bit."""
import numpy as np
import pytest

from paper_2508_07423_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["ETX_FP32", "ETX_BF16", "ETX_FP8_E4M3"])
@pytest.mark.parametrize("name,tracks,products,fuse,compact", [("c1", 3, 1, 0, 0), ("c1", 60, 0, 0, 1), ("c2", 5, 1, 0, 1),
                                                               ("c2", 130, 0, 1, 1), ("c2", 257, 1, 1, 0), ("c3", 64, 1, 1, 1),
                                                               ("c2", 130, 0, 0, 0), ("c2", 600, 0, 0, 0), ("c2", 900, 1, 0, 0),
                                                               ("c3", 257, 0, 0, 1)])
def test_event_alone_and_in_a_batch(name, tracks, products, fuse, compact, precision):
    from paper_2508_07423_amd import etx
    w = synth.WORKLOADS[name].with_(gnn_steps=3, tracks=("fixed", tracks))
    weights = synth.xavier_weights(w)
    events = -(-17000 // (tracks * 9)) if tracks < 100 else 24
    batch = synth.generate_batch(w, events, first=3)
    b = etx.to_device(batch)
    assert b.n_hits > 16384
    p = etx.Pipeline(w, weights, precision=getattr(etx, precision))
    for key, value in (("EDGE_PRODUCTS", products), ("FUSE_MESSAGES", fuse), ("COMPACT_STATE", compact)):
        etx.etx_set_option(p.ctx, getattr(etx, "ETX_OPT_" + key), value)
    if precision == "ETX_FP8_E4M3":
        p.calibrate(b)
    p.run(b)
    whole = p.results(b)
    ho, eo = batch["hit_off"], whole["edge_off"]
    # the first event: its edges lie alike in the 16-edge tiles whose partial sums the messages are made of
    n, m = int(ho[1]), int(eo[1])
    assert n <= 16384
    d = etx.to_device(dict(synth.event_slice(batch, 0), hit_off=np.array([0, n], np.int64)))
    p.run(d)
    one = p.results(d)
    p.close()
    for key in ("src", "dst", "score"):
        assert np.array_equal(one[key].view(np.int32), whole[key][:m].view(np.int32)), key
    assert np.array_equal(one["labels"], whole["labels"][:n])
