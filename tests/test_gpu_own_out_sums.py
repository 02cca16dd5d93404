"""The node kernel's own out-sums (sparse graphs, compact state) against the
edge kernels' tile reductions: the same bits, for rows of every length up to
k_max and every position relative to the 16-edge tiles."""
import numpy as np
import pytest

from paper_2508_07423_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# radii: about 1 and about 4 edges per hit on average (own sums), and above the rule (edge kernels' sums)
@pytest.mark.parametrize("precision", ["bf16", "fp8"])
@pytest.mark.parametrize("radius,low,high", [(0.022, 0.3, 2.5), (0.031, 2.5, 6.0), (0.06, 6.0, 64.0)])
def test_own_out_sums_same_bits(radius, low, high, precision):
    from paper_2508_07423_amd import etx
    w = synth.C3.with_(k_max=64, radius=radius)
    batch = synth.generate_batch(w.with_(tracks=("fixed", 300)), 3, first=5)
    weights = synth.xavier_weights(w)
    b = etx.to_device(batch)
    out = []
    for fuse in (0, 1):
        p = etx.Pipeline(w, weights, precision=etx.ETX_BF16 if precision == "bf16" else etx.ETX_FP8_E4M3)
        etx.etx_set_option(p.ctx, etx.ETX_OPT_COMPACT_STATE, 1)
        etx.etx_set_option(p.ctx, etx.ETX_OPT_FUSE_MESSAGES, fuse)
        if precision == "fp8":
            p.calibrate(b)
        p.run(b)
        res = p.results(b)
        h = p.view(b, etx.ETX_VIEW_NODE_H, torch.int16).cpu().numpy()[:b.n_hits * w.gnn_hidden]
        p.close()
        out.append((res["src"], res["dst"], res["score"].view(np.int32), res["labels"], h))
    rows = np.bincount(out[0][0], minlength=b.n_hits)
    assert low <= rows.mean() < high, rows.mean()
    if low >= 2.5:
        assert rows.max() >= 17
        assert len(np.unique(rows[rows > 0])) >= 17       # run lengths 1 to 16 and longer
    for x, y in zip(*out):
        assert np.array_equal(x, y)
