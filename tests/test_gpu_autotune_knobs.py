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
