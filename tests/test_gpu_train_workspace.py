"""The training workspace holds gradient partials for the rows there can be: a
handful of hits does not take a full set, and steps whose workspace ends where
the size call says give the gradients of a roomy one and write nothing past it."""
import numpy as np
import pytest

from paper_2508_07423_amd import synth
from tests.test_gpu_train_sizes import _mods, _setup

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GUARD = 1 << 20


def _steps(w, tracks, events, capacity):
    """Gradients of the embedding and network steps, with guard bytes after the workspace."""
    etx, T, tr, batch, b, truth, ts, keep = _setup(w, synth.xavier_weights(w), events)
    if capacity is not None:
        allocate = tr.allocate
        tr.allocate = lambda bb, cap=None: allocate(bb, capacity)
    tr.allocate_train(b)
    room = tr.tws_bytes
    tr.tws = torch.full((room + 256 + GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
    tr.tws_ptr = (tr.tws.data_ptr() + 255) & ~255
    n_emb = sum(W.size + v.size for W, v in synth.xavier_weights(w)["emb"])
    tr.embed_step(b, ts, 0.1, 3.0, w.radius, 0.0, 1)
    emb = tr.gradient(b)[:n_emb]
    tr.gnn_step(b, ts, 0.25, 2.0, 0.0, 1)
    net = tr.gradient(b)[n_emb:]
    edges = int(tr.iview(b, etx.ETX_VIEW_ROW_PTR, torch.int64)[-1].item())
    past = tr.tws_ptr - tr.tws.data_ptr() + room
    assert (tr.tws[past:] == 0xA5).all()
    tr.close()
    return emb, net, edges, room, b.n_hits


# twelve hits; a few more edges than hits; more rows than partials
@pytest.mark.parametrize("tracks,events", [(1, 1), (3, 1), (10, 1), (40, 2)])
def test_tight_workspace(tracks, events):
    w = synth.C3.with_(tracks=("fixed", tracks), gnn_steps=2)
    emb, net, edges, room, hits = _steps(w, tracks, events, None)
    tight = _steps(w, tracks, events, edges + 8)
    assert tight[2] == edges and tight[3] <= room
    np.testing.assert_array_equal(tight[0], emb)
    np.testing.assert_array_equal(tight[1], net)


def test_few_hits_take_few_partials():
    w = synth.C2
    etx, T = _mods()
    tr = T.Trainer(w, synth.xavier_weights(w))
    H = w.gnn_hidden
    full = 256 * 4 * 8 * 2 * (4 * H * H + 2 * H)          # all partials of the message-passing networks alone
    few, many = (etx.etx_train_workspace_size(tr.ctx, 1, n, 64 * n) for n in (12, 2500))
    assert few < full / 2 and many > full
    tri = [etx.etx_train_triplet_workspace_size(tr.ctx, 1, 12, 66, n) for n in (20, 4000)]
    per_triplet = 4 * etx.ETX_TRIPLET_NPARAM(H)
    assert tri[1] - tri[0] > 200 * per_triplet
    tr.close()
