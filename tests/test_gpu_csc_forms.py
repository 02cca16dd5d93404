"""The (dst, src) permutation where its workgroups change form within a batch:
a large sparse event among many small ones, columns as long as the event, and
large events of few edges in batches of any size.  The permutation is compared
with numpy's; a form that does not suit its event is told from the stage times
of two batches of the same run."""
import numpy as np
import pytest

from paper_2508_07423_amd import synth
from tests.test_gpu_graph_sizes import MANY, _batch, _event

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _csc_ms(etx, p, b, cap=None):
    """Time of the CSC stage: the best of five runs."""
    etx.etx_set_option(p.ctx, etx.ETX_OPT_PROFILE, 1)
    best = np.inf
    for _ in range(6):
        etx.etx_profile_reset(p.ctx)
        p.run(b, cap)
        best = min(best, etx.etx_profile_read(p.ctx)["csc"][0])
    etx.etx_set_option(p.ctx, etx.ETX_OPT_PROFILE, 0)
    return best


def _check_permutation(etx, p, b, batch):
    res = p.results(b)
    order = np.lexsort((res["src"], res["dst"]))
    assert np.array_equal(p.view(b, etx.ETX_VIEW_CSC_EDGE, torch.int32).cpu().numpy()[:len(order)], order)
    assert np.array_equal(p.view(b, etx.ETX_VIEW_COL_PTR, torch.int64).cpu().numpy(),
                          np.searchsorted(res["dst"][order], np.arange(b.n_hits + 1)))
    return res


def test_large_sparse_event_among_small_ones():
    """One event of 16,384 hits takes about as long among 300 small ones as alone: at most twice the passes over its
    edges (half the LDS), where one wave walking its rows takes an order of magnitude longer."""
    from paper_2508_07423_amd import etx
    w = synth.C1.with_(k_max=6, gnn_steps=1)
    p = etx.Pipeline(w, synth.xavier_weights(w))
    alone, among = (_csc_ms(etx, p, etx.to_device(_batch(s))) for s in ([16384], MANY + [16384]))
    p.close()
    assert among < 3 * alone, (among, alone)


def _hub_event(n, targets):
    """n hits on two planes, `targets` of them on the second: columns of about n / targets edges."""
    ev = _event(n, 5)
    ev["plane"] = np.where(np.arange(n) % max(n // targets, 1) == 0, 1, 0).astype(np.int32)
    while ev["plane"].sum() > targets:
        ev["plane"][np.flatnonzero(ev["plane"])[-1]] = 0
    return ev


# columns of 400 edges and of about half the LDS (8,192); one column of nearly the whole event
@pytest.mark.parametrize("place", [0, 1])
@pytest.mark.parametrize("n,targets", [(9000, 20), (16384, 40), (16384, 2), (12000, 1), (16384, 1), (4097, 1)])
def test_long_columns(n, targets, place):
    from paper_2508_07423_amd import etx
    w = synth.C1.with_(k_max=1, radius=50.0, gnn_steps=1)
    small, hub = _batch(MANY), _hub_event(n, targets)
    batch = {k: np.concatenate([small[k], hub[k]]) for k in hub}
    batch["hit_off"] = np.concatenate([small["hit_off"], [small["hit_off"][-1] + n]])
    b = etx.to_device(batch)
    p = etx.Pipeline(w, synth.xavier_weights(w))
    etx.etx_set_option(p.ctx, etx.ETX_OPT_CSC_PLACE, place)
    p.run(b)
    res = _check_permutation(etx, p, b, batch)
    p.close()
    columns = np.bincount(res["dst"], minlength=b.n_hits)[-n:]
    assert columns.max() >= (n - targets) // targets


def test_short_rows_walk_by_edges():
    """Without placing, a walked event of few edges takes time with its edges, not its rows: with k_max 2 it has less
    than half the edges of k_max 6."""
    from paper_2508_07423_amd import etx
    batch = _batch([16384, 16384])
    b = etx.to_device(batch)
    ms, edges = [], []
    for k_max in (2, 6):
        w = synth.C1.with_(k_max=k_max, gnn_steps=1)
        p = etx.Pipeline(w, synth.xavier_weights(w))
        etx.etx_set_option(p.ctx, etx.ETX_OPT_CSC_PLACE, 0)
        ms.append(_csc_ms(etx, p, b))
        edges.append(len(_check_permutation(etx, p, b, batch)["src"]))
        p.close()
    assert edges[0] < 0.5 * edges[1]
    assert ms[0] < 0.75 * ms[1], ms


# events on both sides of 2,048 hits and of four edges per hit
@pytest.mark.parametrize("sizes,k_max", [([2048, 2049, 2050], 3), ([2049, 4100, 0, 63], 4), ([16384, 8193], 5),
                                         ([4096, 2500], 9), ([16384], 1)])
def test_short_rows_walked(sizes, k_max):
    from paper_2508_07423_amd import etx
    w = synth.C1.with_(k_max=k_max, gnn_steps=1)
    batch = _batch(sizes)
    b = etx.to_device(batch)
    p = etx.Pipeline(w, synth.xavier_weights(w))
    etx.etx_set_option(p.ctx, etx.ETX_OPT_CSC_PLACE, 0)
    p.run(b)
    _check_permutation(etx, p, b, batch)
    p.close()


def test_small_dense_events_are_not_sorted_in_memory():
    """800 events of about twelve edges per hit: the choice by row length is no slower than walking every event, which
    takes them all in wide workgroups (half as much again allowed; sorting their columns in memory took 2.5 times)."""
    from paper_2508_07423_amd import etx
    w = synth.C1.with_(gnn_steps=1)
    batch = synth.generate_batch(w, 800, first=1)
    b = etx.to_device(batch)
    p = etx.Pipeline(w, synth.xavier_weights(w))
    p.run(b)
    per_hit = len(_check_permutation(etx, p, b, batch)["src"]) / b.n_hits
    assert 8 < per_hit < 16, per_hit
    ms = []
    for place in (0, 1):
        etx.etx_set_option(p.ctx, etx.ETX_OPT_CSC_PLACE, place)
        ms.append(_csc_ms(etx, p, b))
    p.close()
    assert ms[1] < 1.6 * ms[0], ms


# events on both sides of six edges per hit in one batch of more events than CUs, up to 4,096 hits and above
@pytest.mark.parametrize("k_max", [5, 6, 7, 8, 12])
def test_rows_around_the_sorted_length(k_max):
    from paper_2508_07423_amd import etx
    w = synth.C1.with_(k_max=k_max, gnn_steps=1)
    batch = _batch(MANY + [2000, 4095, 4096, 4097, 700, 0, 1])
    b = etx.to_device(batch)
    p = etx.Pipeline(w, synth.xavier_weights(w))
    p.run(b)
    _check_permutation(etx, p, b, batch)
    p.close()


def test_many_small_sparse_events_walked():
    """Without placing, 4,000 events of two edges per hit take at most three times as long as placed (four times in
    workgroups as large as the CU)."""
    from paper_2508_07423_amd import etx
    w = synth.C1.with_(k_max=2, gnn_steps=1)
    few = [_event(490, i) for i in range(8)]
    batch = {k: np.concatenate([few[i % 8][k] for i in range(4000)]) for k in few[0]}
    batch["hit_off"] = np.arange(4001, dtype=np.int64) * 490
    b = etx.to_device(batch)
    p = etx.Pipeline(w, synth.xavier_weights(w))
    ms = []
    for place in (0, 1):
        etx.etx_set_option(p.ctx, etx.ETX_OPT_CSC_PLACE, place)
        ms.append(_csc_ms(etx, p, b))
        _check_permutation(etx, p, b, batch)
    p.close()
    assert ms[0] < 3 * ms[1], ms


# events on both sides of 1,024 hits and of four edges per hit, in batches above and below 1,024 hits per event
@pytest.mark.parametrize("k_max", [1, 4, 5, 6])
@pytest.mark.parametrize("extra", [[1023, 1024, 1025, 0, 63, 1, 16384], [4097] * 100])
def test_small_events_walked(extra, k_max):
    from paper_2508_07423_amd import etx
    w = synth.C1.with_(k_max=k_max, gnn_steps=1)
    batch = _batch(MANY + extra)
    b = etx.to_device(batch)
    p = etx.Pipeline(w, synth.xavier_weights(w))
    etx.etx_set_option(p.ctx, etx.ETX_OPT_CSC_PLACE, 0)
    p.run(b)
    _check_permutation(etx, p, b, batch)
    p.close()
