"""Training gradients against the FP64 oracle at the sizes where the row
kernels can go wrong: fewer rows than chunks, chunks of one tile with a
remainder, chunks of several tiles, an event without edges, both hidden sizes,
every embedding width with the fewest and the most layers and the narrowest and
widest output.  Bounds as in test_gpu_train (the embedding's by layer); the
graph is the step's own."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2508_07423_amd import synth
from tests.test_gpu_train import _bound, _embedding_abs_terms, _gnn_param_offset, _mods

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _setup(w, weights, events):
    etx, T = _mods()
    batch = synth.generate_batch(w, events, first=3)
    tr = T.Trainer(w, weights)
    truth = T.truth_arrays(batch, w, np.random.default_rng(0))
    ts, keep = T.truth_to_device(truth)
    return etx, T, tr, batch, etx.to_device(batch), truth, ts, keep


def _edges(etx, tr, b):
    E = int(tr.iview(b, etx.ETX_VIEW_ROW_PTR, torch.int64)[-1].item())
    return tr.src[:E].cpu().numpy(), tr.dst[:E].cpu().numpy()


# (workload, tracks per event, events, message-passing steps, least edges): 12 hits; 256 chunks of 2 rows; chunks of
# more than one 64-row tile (over 16,384 edges) with both hidden sizes; one plane, no edges
@pytest.mark.parametrize("name,tracks,events,steps,least", [
    ("c3", 1, 1, 4, 1), ("c1", 30, 1, 1, 256), ("c3", 60, 2, 1, 16385), ("c2", 80, 1, 1, 16385), ("c3", 8, 1, 2, 0)])
def test_network_gradient_at_row_counts(name, tracks, events, steps, least):
    w = synth.WORKLOADS[name].with_(tracks=("fixed", tracks), gnn_steps=steps)
    if least == 0:
        w = w.with_(radius=1e-6)
    weights = synth.xavier_weights(w)
    etx, T, tr, batch, b, truth, ts, keep = _setup(w, weights, events)
    loss = float(tr.gnn_step(b, ts, 0.25, 2.0, 0.0, 1).item())
    o = _gnn_param_offset(w)
    g = tr.gradient(b)[o:]
    src, dst = _edges(etx, tr, b)
    tr.close()
    if least == 0:
        assert len(src) == 0 and loss == 0 and not g.any()
        return
    assert len(src) >= least
    lab = (truth["succ"][src] == dst).astype(np.uint8)
    _, cart = O.features(batch["x"], batch["y"], batch["z"], w.r_scale, w.z_scale)
    lo, go = O.gnn_focal_loss_grad(cart, src, dst, weights, w.gnn_hidden, w.gnn_steps, lab, 0.25, 2.0)
    cp = cart * (1 + 2.0 ** -23 * np.random.default_rng(3).standard_normal(cart.shape))
    spread = np.abs(O.gnn_focal_loss_grad(cp, src, dst, weights, w.gnn_hidden, w.gnn_steps, lab, 0.25, 2.0)[1] - go)
    err = np.abs(g - go)
    assert abs(loss - lo) <= 1e-5 * abs(lo)
    assert np.all(err <= _bound(go, spread)), err.max()


@pytest.mark.parametrize("width,layers,dim,tracks", [(32, 1, 4, 1), (32, 4, 16, 40), (64, 3, 12, 40), (128, 1, 16, 40),
                                                     (128, 4, 4, 40), (64, 2, 8, 1500)])
def test_embedding_gradient_at_shapes(width, layers, dim, tracks):
    """1500 tracks in one ten-plane event: 15,000 hits, chunks of 59 rows."""
    w = synth.C1.with_(tracks=("fixed", tracks), emb_hidden=width, emb_layers=layers, emb_dim=dim, k_max=8)
    weights = synth.xavier_weights(w)
    etx, T, tr, batch, b, truth, ts, keep = _setup(w, weights, 1)
    margin, r_train = 16.0, 0.02         # every fake pair is inside the margin: no kink
    loss = float(tr.embed_step(b, ts, margin, 3.0, r_train, 0.0, 1).item())
    n_emb = _gnn_param_offset(w)
    g = tr.gradient(b)[:n_emb]
    src, dst = _edges(etx, tr, b)
    tr.close()
    succ, rnd, q = truth["succ"], truth["rnd"], truth["query"].astype(bool)
    qi = np.nonzero(q & (succ >= 0))[0]
    hard = q[src] & (truth["particle"][dst] >= 0) & (dst != succ[src])
    rq = np.nonzero(q & (rnd >= 0) & (rnd != succ))[0]
    gen = (qi.astype(np.int32), succ[qi])
    fake = (np.concatenate([src[hard], rq]).astype(np.int32), np.concatenate([dst[hard], rnd[rq]]).astype(np.int32))
    cyl, _ = O.features(batch["x"], batch["y"], batch["z"], w.r_scale, w.z_scale)
    L64 = [(W.astype(np.float64), v.astype(np.float64)) for W, v in weights["emb"]]
    emb = O.embed(cyl, weights["emb"])
    assert (((emb[fake[0]] - emb[fake[1]]) ** 2).sum(1) < 0.999 * margin).all()
    lo, go = O.embed_hinge_loss_grad(cyl, L64, gen, fake, margin, 3.0)
    cp = cyl * (1 + 2.0 ** -23 * np.random.default_rng(4).standard_normal(cyl.shape))
    spread = np.abs(O.embed_hinge_loss_grad(cp, L64, gen, fake, margin, 3.0)[1] - go)
    S = _embedding_abs_terms(cyl, L64, gen, fake, margin, 3.0)
    assert abs(loss - lo) <= 1e-5 * abs(lo)
    # Layer by layer in the 2-norm: a hidden value just above its ReLU has a large relative error, so single
    # weights of it do too, but no layer as a whole.
    norm, at = np.linalg.norm, 0
    for W, v in weights["emb"]:
        part = slice(at, at + W.size + v.size)
        at = part.stop
        bound = 1e-4 * norm(go[part]) + 16 * np.log2(len(cyl)) * 2.0 ** -24 * norm(S[part]) + 4 * norm(spread[part])
        assert norm(g[part] - go[part]) <= bound, (W.shape, norm(g[part] - go[part]), bound)
