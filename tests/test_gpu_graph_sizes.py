"""Plane bucketing, row offsets and the (dst, src) permutation at the event and
batch sizes where their kernels change form: the small and the wide CSC
workgroups (4,096 hits, one event per CU), row ranges of the largest event,
placement over several column ranges, one to seventeen scan blocks,
shuffled hits.  All are whole numbers with one right answer, formed with numpy
from the run's own edges."""
import numpy as np
import pytest

from paper_2508_07423_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _event(n, seed):
    """n hits of the ten-plane detector in random order."""
    w = synth.C1.with_(tracks=("fixed", max(1, n // 8 + 2)), hit_order="shuffled")
    ev = synth.generate_event(w, seed, seed_space=31)
    while len(ev["x"]) < n:
        more = synth.generate_event(w, seed + 1000, seed_space=31)
        ev = {k: np.concatenate([ev[k], more[k]]) for k in ev}
    return {k: v[:n] for k, v in ev.items()}


def _batch(sizes):
    evs = [_event(n, i) for i, n in enumerate(sizes)]
    out = {k: np.concatenate([e[k] for e in evs]) for k in evs[0]}
    out["hit_off"] = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    return out


MANY = [17 + (i * 37) % 90 for i in range(300)]


# (event sizes, k_max, least edges per hit of the largest event): k_max 32 gives long rows, 6 short ones
@pytest.mark.parametrize("place", [0, 1])
@pytest.mark.parametrize("sizes,k_max,least", [
    ([1], 32, 0), ([0, 63, 0, 64, 65, 0], 32, 0), ([4096], 6, 2), ([4097, 5], 6, 2), ([4096, 4097], 32, 16),
    ([8192], 6, 2), ([8193], 32, 16), ([16384], 32, 16), ([16384], 6, 2), ([8192, 8193], 32, 16), (MANY, 32, 0),
    (MANY + [4097, 0, 4500], 6, 2), ([16384, 16384, 1], 6, 2), ([16384] * 8, 6, 2), ([16384] * 8 + [3, 0], 6, 2),
    (MANY + [8192, 8193], 6, 2), (MANY + [16384], 6, 2), (MANY + [16384, 4097], 32, 16)])
def test_graph_kernels_at_sizes(sizes, k_max, least, place):
    from paper_2508_07423_amd import etx
    w = synth.C1.with_(k_max=k_max)
    batch = _batch(sizes)
    b = etx.to_device(batch)
    p = etx.Pipeline(w, synth.xavier_weights(w))
    etx.etx_set_option(p.ctx, etx.ETX_OPT_CSC_PLACE, place)
    p.run(b)
    res = p.results(b)
    E, n, ho = len(res["src"]), b.n_hits, batch["hit_off"]
    src, dst = res["src"], res["dst"]
    view = lambda which, dt: p.view(b, which, dt).cpu().numpy()
    bucket, po = view(etx.ETX_VIEW_BUCKET, torch.int32), view(etx.ETX_VIEW_PLANE_OFF, torch.int32)
    row_ptr, col_ptr = view(etx.ETX_VIEW_ROW_PTR, torch.int64), view(etx.ETX_VIEW_COL_PTR, torch.int64)
    csc = view(etx.ETX_VIEW_CSC_EDGE, torch.int32)[:E]
    p.close()
    event = np.repeat(np.arange(len(sizes)), sizes)
    assert np.array_equal(bucket, np.lexsort((np.arange(n), batch["plane"], event)))
    counts = np.zeros((len(sizes), w.n_planes + 1), np.int32)
    np.add.at(counts, (event, batch["plane"] + 1), 1)
    assert np.array_equal(po.reshape(counts.shape), np.cumsum(counts, 1))
    assert np.array_equal(row_ptr, np.searchsorted(src, np.arange(n + 1)))
    assert np.array_equal(res["edge_off"], row_ptr[ho])
    order = np.lexsort((src, dst))
    assert np.array_equal(csc, order)
    assert np.array_equal(col_ptr, np.searchsorted(dst[order], np.arange(n + 1)))
    big = int(np.argmax(sizes))
    per_hit = (row_ptr[ho[big + 1]] - row_ptr[ho[big]]) / max(sizes[big], 1)
    assert per_hit >= least, per_hit


@pytest.mark.parametrize("sizes,kept", [
    ([300], "all"), ([300], "few"), ([4096], "all"), ([4097], "few"), ([4097], "all"), ([16384, 0, 7], "few"),
    (MANY, "all"), (MANY + [4097, 0, 4500], "few"), (MANY + [4097, 0, 4500], "all")])
def test_components_at_sizes(sizes, kept):
    """Component labels when every edge is kept and when about a fifth is."""
    from oracle import oracle as O
    from paper_2508_07423_amd import etx
    batch = _batch(sizes)
    b = etx.to_device(batch)
    w = synth.C1.with_(k_max=8)
    weights = synth.xavier_weights(w)
    p = etx.Pipeline(w, weights)
    p.run(b)
    score = p.results(b)["score"]
    p.close()
    thr = float(np.float32(score.min() if kept == "all" else np.quantile(score, 0.8)))
    p = etx.Pipeline(w.with_(threshold=thr), weights)
    p.run(b)
    res = p.results(b)
    p.close()
    keep = res["score"] >= np.float32(thr)
    share = keep.mean()
    assert share == 1 if kept == "all" else 0.1 < share < 0.3
    assert np.array_equal(res["labels"], O.components(b.n_hits, res["src"], res["dst"], keep))


@pytest.mark.parametrize("sizes", [[300], [8192, 1], [9000, 9000, 0], [16384] * 8, [16384] * 8 + [1]])
def test_too_many_edges_at_sizes(sizes):
    """One edge more than fits is reported with the need, whichever form the scan has; the need itself fits."""
    from paper_2508_07423_amd import etx
    w = synth.C1.with_(k_max=6, gnn_steps=1)
    b = etx.to_device(_batch(sizes))
    p = etx.Pipeline(w, synth.xavier_weights(w))
    p.run(b)
    need = len(p.results(b)["src"])
    assert need > 0
    p.run(b, need - 1)
    torch.cuda.synchronize()
    st = p.status.cpu().numpy()
    assert st[0] == etx.ETX_ERR_CAPACITY and st[1] == need
    p.run(b, need)
    assert len(p.results(b)["src"]) == need
    p.close()
