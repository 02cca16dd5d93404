"""What the autotuner's knobs are judged by, and which it leaves alone."""
import json

import pytest

from paper_2508_07423_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _tune(w, tracks, events, precision, compact, tmp_path, before=()):
    """Tunes a batch; returns the record's choice, the options in effect before and after, and the batch's hits."""
    from paper_2508_07423_amd import etx
    batch = synth.generate_batch(w.with_(tracks=("fixed", tracks)), events, first=3)
    b = etx.to_device(batch)
    p = etx.Pipeline(w, synth.trained_weights(w), precision=getattr(etx, precision))
    for key, value in (("COMPACT_STATE", compact),) + tuple(before):
        etx.etx_set_option(p.ctx, getattr(etx, "ETX_OPT_" + key), value)
    if precision == "ETX_FP8_E4M3":
        p.calibrate(b)
    log = tmp_path / "trials.jsonl"
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        out = p.allocate(b, 8 * b.n_hits)
        etx.etx_autotune(p.ctx, p.hits_struct(b), out, p.ws_ptr, p.ws_bytes, s.cuda_stream, str(log))
    table = tmp_path / "tuning.txt"
    etx.etx_tuning_save(p.ctx, str(table))
    entry = dict(kv.split("=") for kv in table.read_text().splitlines()[-1].split()[3:])
    p.close()
    return json.loads(log.read_text())["choice"], {int(k): int(v) for k, v in entry.items()}, b.n_hits


@pytest.mark.parametrize("name,precision,compact,edges", [("c3", "ETX_BF16", 1, True), ("c3", "ETX_FP8_E4M3", 1, True),
                                                          ("c3", "ETX_BF16", 0, False), ("c3", "ETX_FP32", 1, False),
                                                          ("c2", "ETX_BF16", 1, False)])
def test_fused_messages_are_judged_by_what_they_change(name, precision, compact, edges, tmp_path):
    """With the compact state of hidden size 32 the edge kernels' out-sums depend on the knob: their stages count, and
    the edge kernels' own knobs come after it."""
    choice, _, _ = _tune(synth.WORKLOADS[name], 100, 8, precision, compact, tmp_path)
    stages = set(choice["fuse_messages_stages"])
    assert stages == {"segsum", "node_step"} | ({"edge_encode", "edge_step"} if edges else set())
    order = list(choice)
    assert order.index("fuse_messages") < order.index("edge_threads_x_wg_per_cu")
    assert order.index("fuse_messages") < order.index("edge_pipeline")


@pytest.mark.parametrize("name,tracks,events,small", [("c1", 50, 1, True), ("c3", 100, 8, True), ("c3", 100, 24, False)])
def test_unroll_is_tuned_where_it_is_used(name, tracks, events, small, tmp_path):
    """Batches of up to 16,384 hits keep eight rows in flight whatever the option, and fused runs launch no message
    sums: no trials, and the stored entry holds the default."""
    from paper_2508_07423_amd import etx
    choice, entry, hits = _tune(synth.WORKLOADS[name], tracks, events, "ETX_FP32", 0, tmp_path, [("SEGSUM_UNROLL", 1)])
    assert (hits <= 16384) == small
    if small or choice["fuse_messages"] == "1":
        assert "segsum_unroll" not in choice and entry[etx.ETX_OPT_SEGSUM_UNROLL] == 4
    else:
        assert int(choice["segsum_unroll"]) == entry[etx.ETX_OPT_SEGSUM_UNROLL]
    assert "radius_sort_min" in choice
