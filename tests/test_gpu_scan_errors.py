"""A batch with more edges than its capacity, at the sizes where the row-offset
scan is one workgroup, two and sixteen, which run side by side while one of
them reports the error: the need is reported and the event offsets are left as
they were, as for batches above those sizes; also after an input error, when
the scan has nothing to do."""
import numpy as np
import pytest

from paper_2508_07423_amd import synth
from tests.test_gpu_graph_sizes import _batch

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sizes", [[300], [8192, 1], [16384] * 8, [40] * 3000, [16384] * 8 + [1]])
def test_offsets_untouched_on_error(sizes):
    from paper_2508_07423_amd import etx
    w = synth.C1.with_(k_max=6, gnn_steps=1)
    b = etx.to_device(_batch(sizes))
    p = etx.Pipeline(w, synth.xavier_weights(w))
    p.run(b)
    need = len(p.results(b)["src"])
    p.allocate(b, need - 1)
    for _ in range(20):
        p.edge_off.fill_(-7)
        p.run(b, need - 1)
        torch.cuda.synchronize()
        st = p.status.cpu().numpy()
        assert st[0] == etx.ETX_ERR_CAPACITY and st[1] == need
        assert (p.edge_off == -7).all()
    plane = b.plane.clone()
    b.plane[-1] = w.n_planes
    p.edge_off.fill_(-7)
    p.run(b, need - 1)
    torch.cuda.synchronize()
    assert p.status.cpu().numpy()[0] == etx.ETX_ERR_INPUT and (p.edge_off == -7).all()
    b.plane.copy_(plane)
    p.run(b, need)
    assert len(p.results(b)["src"]) == need
    p.close()
