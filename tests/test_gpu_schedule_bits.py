"""Launch schedules that give the same bits, at batches where each of their
forms runs: the message sums' rows in flight on batches that follow the option,
the small node update against the large one at both hidden sizes, and the node
kernel's own out-sums as production runs them (edge products in the edge
kernels, pruned graphs)."""
import numpy as np
import pytest

from paper_2508_07423_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KEYS = ("src", "dst", "score", "labels")


def _runs(w, weights, batch, precision, variants, prefilter=None):
    """The outputs (bits) of one batch under each set of options."""
    from paper_2508_07423_amd import etx
    b = etx.to_device(batch)
    out = []
    for options in variants:
        p = etx.Pipeline(w, weights, precision=getattr(etx, precision))
        for key, value in options.items():
            etx.etx_set_option(p.ctx, getattr(etx, "ETX_OPT_" + key), value)
        if precision == "ETX_FP8_E4M3":
            p.calibrate(b)
        if prefilter is not None:
            params, tau = prefilter
            etx.etx_prefilter_set(p.ctx, params)
            etx.etx_prefilter_config(p.ctx, 1, tau)
        p.run(b)
        res = p.results(b)
        prob = p.view(b, etx.ETX_VIEW_PF_PROB, torch.float32).cpu().numpy() if prefilter is not None else None
        p.close()
        out.append(dict({k: res[k].view(np.int32) for k in KEYS}, prob=prob))
    return b, out


def _same(out):
    for other in out[1:]:
        for k in KEYS:
            assert np.array_equal(out[0][k], other[k]), k


# sparse and dense rows at both hidden sizes
@pytest.mark.parametrize("precision,compact", [("ETX_FP32", 0), ("ETX_BF16", 1), ("ETX_FP8_E4M3", 1)])
@pytest.mark.parametrize("name,radius,tracks,events", [("c3", 0.022, 100, 24), ("c3", 0.1, 100, 24), ("c2", 0.03, 100, 24),
                                                       ("c2", 0.12, 100, 24)])
def test_unroll_same_bits(name, radius, tracks, events, precision, compact):
    w = synth.WORKLOADS[name].with_(radius=radius, gnn_steps=2, tracks=("fixed", tracks))
    batch = synth.generate_batch(w, events, first=3)
    b, out = _runs(w, synth.xavier_weights(w), batch, precision,
                   [dict(SEGSUM_UNROLL=u, FUSE_MESSAGES=0, COMPACT_STATE=compact) for u in (1, 2, 4, 8)])
    assert b.n_hits > 16384                      # smaller ones keep eight rows whatever the option
    _same(out)


@pytest.mark.parametrize("name,tracks,products", [("c1", 3, 1), ("c1", 60, 0), ("c3", 64, 1), ("c3", 257, 0), ("c2", 130, 0),
                                                  ("c2", 5, 1)])
def test_small_node_update_same_bits(name, tracks, products):
    """FP32, messages not fused: an event alone takes the form with a workgroup per 16 hits, the batch the large one."""
    from paper_2508_07423_amd import etx
    w = synth.WORKLOADS[name].with_(gnn_steps=3, tracks=("fixed", tracks))
    limit = (2 if w.gnn_hidden == 64 else 8) * 16 * torch.cuda.get_device_properties(0).multi_processor_count
    first = synth.generate_batch(w, 1, first=3)
    batch = synth.generate_batch(w, int(1.3 * limit / len(first["x"])) + 1, first=3)
    assert len(first["x"]) <= limit < len(batch["x"])
    weights, options = synth.xavier_weights(w), [dict(EDGE_PRODUCTS=products, FUSE_MESSAGES=0)]
    _, (whole,) = _runs(w, weights, batch, "ETX_FP32", options)
    _, (one,) = _runs(w, weights, first, "ETX_FP32", options)
    m, n = len(one["src"]), len(first["x"])
    for k in ("src", "dst", "score"):
        assert np.array_equal(one[k], whole[k][:m]), k
    assert np.array_equal(one["labels"], whole["labels"][:n])


@pytest.mark.parametrize("precision", ["ETX_BF16", "ETX_FP8_E4M3"])
@pytest.mark.parametrize("products", [0, 1])
@pytest.mark.parametrize("pruned", [False, True])
def test_own_out_sums_in_production_schedules(precision, products, pruned):
    """Fused against unfused messages, with the products in either kernel, whole graphs and pruned ones."""
    w = synth.C3.with_(k_max=64, radius=0.031, tracks=("fixed", 300))
    batch = synth.generate_batch(w, 3, first=5)
    rng = np.random.default_rng(3)
    params = np.concatenate([np.concatenate([W.ravel(), rng.normal(0, 0.1, v.shape).ravel()])
                             for W, v in synth.xavier_prefilter(3)]).astype(np.float32)
    variants = [dict(FUSE_MESSAGES=f, EDGE_PRODUCTS=products, COMPACT_STATE=1) for f in (0, 1)]
    prefilter = None
    if pruned:                                   # tau at the median probability: half of the candidates go
        _, (o,) = _runs(w, synth.xavier_weights(w), batch, "ETX_FP32", [{}], (params, 0.0))
        prefilter = (params, float(np.median(o["prob"][:len(o["src"])])))
    b, out = _runs(w, synth.xavier_weights(w), batch, precision, variants, prefilter)
    per_hit = len(out[0]["src"]) / b.n_hits
    assert 1.0 < per_hit < 6.0, per_hit          # the node kernel's sums
    _same(out)
