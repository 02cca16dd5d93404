"""The performance cases of the track-finding library: the calls a program
makes, over the range of sizes, precisions and options it makes them with.

A case is a dict of plain values.  ``call`` names the entry point:

  run              Pipeline.run (etx_run): the whole pipeline on a packed batch
  tracks           Pipeline.run_tracks (etx_run_tracks): the pipeline and the triplet stage
  train_embed      Trainer.embed_step: one training step of the embedding
  train_gnn        Trainer.gnn_step: one training step of the interaction network
  train_triplets   Trainer.triplet_step: the same with the triplet term
  train_prefilter  Pipeline.prefilter_train_step: one training step of the edge prefilter

``workload`` is one of the package's workloads (detector geometry, event
recipe, network sizes), ``events`` the batch size, ``tracks`` a fixed number of
tracks per event (0: the workload's own recipe).  ``weights`` are the
workload's random Xavier weights (a dense candidate graph) or its committed
trained ones (two to three candidates per hit).  Online programs replay a
captured HIP graph (``graph``) and use the launch schedule the autotuner found
for their kind of batch (``tuned``).
"""
import math

import numpy as np
import torch

from paper_2508_07423_amd import etx, synth
from paper_2508_07423_amd import prefilter_train
from paper_2508_07423_amd import train as training

PRECISION = {"fp32": etx.ETX_FP32, "bf16": etx.ETX_BF16, "fp8": etx.ETX_FP8_E4M3, "int8": etx.ETX_INT8}

# The schedules the autotuner settles on for dense (random weights) and sparse (trained weights) graphs.
DENSE = dict(EDGE_WG_SIZE=512, EDGE_WG_PER_CU=4, EDGE_PIPELINE=1, NODE_WG_PER_CU=1, FUSE_MESSAGES=1, SEGSUM_UNROLL=4,
             RADIUS_SORT_MIN=1024, RADIUS_FAST=0, XCD_MAP=1, EDGE_PRODUCTS=0, CSC_PLACE=0, RADIUS_SPLIT=1)
SPARSE = dict(EDGE_WG_SIZE=256, EDGE_WG_PER_CU=4, EDGE_PIPELINE=1, NODE_WG_PER_CU=3, FUSE_MESSAGES=1, SEGSUM_UNROLL=4,
              RADIUS_SORT_MIN=128, RADIUS_FAST=1, XCD_MAP=0, EDGE_PRODUCTS=1, CSC_PLACE=1, RADIUS_SPLIT=1)

# hits per event, and candidate edges per hit with random and with trained weights
HITS = {"c1": 490, "c2": 2550, "c3": 1862, "c6": 2040}
EDGES = {"c1": (12.1, 2.0), "c2": (52.3, 2.0), "c3": (26.7, 2.53), "c6": (26.7, 2.74)}
HITS_PER_TRACK = {"c1": 9.8, "c2": 12.75, "c3": 12.75, "c6": 13.6}

# A prefilter that keeps candidates closer than about 0.06 in the embedding (two thirds of them with the trained
# networks): p = sigmoid(SLOPE (CUT - distance)) plus small contributions of the other hidden units.
CUT, SLOPE, TAU = 0.06, 60.0, 0.5
# events whose kept fraction leaves this band run unpruned
BAND = (0.3, 1.0)

# one training step: learning rates and loss parameters of the package's own recipe
LR = {"train_embed": 3e-3, "train_gnn": 2e-3, "train_triplets": 1e-3, "train_prefilter": 1e-2}
W_GEN, ALPHA, GAMMA = 3.0, 0.25, 2.0
POS_WEIGHT = 4.0
# Adam's second moment and step count of a run in progress
MOMENT2, STEP = 1e-4, 500


def _run(name, workload, weights, events, tracks=0, precision="fp32", compact=False, prefilter=False, tuned=False,
         graph=False, call="run"):
    c = dict(call=call, workload=workload, weights=weights, events=events, tracks=tracks, precision=precision,
             compact=compact, prefilter=prefilter, tuned=tuned, graph=graph)
    return c if name is None else dict(c, name=name)


def _train(name, call, workload, weights, events, tracks):
    c = dict(call=call, workload=workload, weights=weights, events=events, tracks=tracks)
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # the smallest call: one event of the ten-plane detector, eager, default options (a first try, a test)
        _run("one-event", "c1", "random", 1, tracks=50),
        # online reconstruction of one full-size event with the trained full-size network: latency
        _run("one-full-event", "c2", "trained", 1, tracks=200, graph=True),
        # the plain pipeline at full size, 1000 events, single precision: the headline throughput
        _run("full-size", "c2", "random", 1000),
        # the full-size network in BF16 with the state stored in BF16, a batch as a trigger farm buffers it
        _run("full-size-bf16", "c2", "random", 100, precision="bf16", compact=True),
        # uneven events (200 to 8000 hits) with a dense graph
        _run("uneven", "c3", "random", 1000, tuned=True, graph=True),
        # production: uneven events, trained network, single precision
        _run("trained", "c3", "trained", 10000, tuned=True, graph=True),
        # production at reduced precision: BF16, compact state, learned prefilter
        _run("trained-bf16-pruned", "c3", "trained", 10000, precision="bf16", compact=True, prefilter=True, tuned=True,
             graph=True),
        # the full method: triplets and tracks that share hits
        _run("tracks", "c6", "trained", 2000, tuned=True, call="tracks"),
        # training, one event per step as the recipe does: embedding, network, network with triplets
        _train("train-embedding", "train_embed", "c3", "trained", 1, 150),
        _train("train-network", "train_gnn", "c3", "trained", 1, 150),
        _train("train-triplets", "train_triplets", "c6", "trained", 1, 150),
        # training of the prefilter, 20 events per step as the recipe does
        _train("train-prefilter", "train_prefilter", "c3", "trained", 20, 0),
    ]


def draw(rng):
    def between(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.random()
    if kind < 0.6:
        workload = rng.choice(["c1", "c2", "c3", "c3"])
        weights = rng.choice(["random", "trained"])
        top = {"c1": 2000, "c2": 600, "c3": 800}[workload] if weights == "random" else \
            {"c1": 10000, "c2": 2000, "c3": 8000}[workload]
        precision, compact = rng.choice([("fp32", False), ("fp32", False), ("bf16", True), ("bf16", False),
                                         ("fp8", True), ("fp8", False), ("int8", False)])
        prefilter = weights == "trained" and workload != "c1" and rng.random() < 0.4
        events = between(1, top)
        tracks = between(20, 600) if events < 40 and rng.random() < 0.5 else 0
        return _run(None, workload, weights, events, tracks, precision, compact, prefilter, rng.random() < 0.5,
                    rng.random() < 0.5)
    if kind < 0.7:
        precision = rng.choice(["fp32", "bf16"])
        return _run(None, "c6", "trained", between(1, 3000), 0, precision, precision == "bf16", False,
                    rng.random() < 0.5, False, call="tracks")
    call = rng.choice(["train_embed", "train_gnn", "train_triplets", "train_prefilter"])
    if call == "train_prefilter":
        return _train(None, call, rng.choice(["c2", "c3"]), "trained", between(2, 60), 0)
    if call == "train_triplets":
        return _train(None, call, "c6", "trained", 1, between(20, 600))
    return _train(None, call, rng.choice(["c2", "c3"]), rng.choice(["random", "trained"]), 1, between(20, 600))


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------

# The detector is symmetric about the beam: a generator event turned by a random angle is another event of the same
# distribution.  A batch holds at most _BASE generator events, each turned by an angle of its own; a larger batch holds
# them again, turned further.  So a case has one number of hits whatever the seed.
_BASE = 200


def _workload(case):
    w = synth.WORKLOADS[case["workload"]]
    return w.with_(tracks=("fixed", float(case["tracks"]))) if case["tracks"] else w


def _events(case, seed):
    """The generator events of the batch, turned, hits in readout order (plane, then azimuth), on the host."""
    n = min(case["events"], _BASE)
    host = synth.generate_batch(_workload(case), n, seed_space=100000)
    off = host.pop("hit_off")
    event = np.repeat(np.arange(n), np.diff(off))
    turn = np.random.default_rng(int(seed)).uniform(0, 2 * math.pi, n)[event]
    x, y = host["x"].astype(np.float64), host["y"].astype(np.float64)
    host["x"] = (np.cos(turn) * x - np.sin(turn) * y).astype(np.float32)
    host["y"] = (np.sin(turn) * x + np.cos(turn) * y).astype(np.float32)
    order = np.lexsort((np.arctan2(host["y"], host["x"]), host["plane"], event))
    return dict({k: v[order] for k, v in host.items()}, hit_off=off)


def _batch(case, seed, host):
    """The batch on the GPU."""
    n = case["events"]
    b = etx.to_device(host)
    base = b.n_events
    if n <= base:
        return b
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    which = torch.arange(n, device="cuda") % base
    turn = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64) * (2 * math.pi)
    turn[:base] = 0
    count = (b.hit_off[1:] - b.hit_off[:-1])[which]
    off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    off[1:] = torch.cumsum(count, 0)
    event = torch.repeat_interleave(torch.arange(n, device="cuda"), count)
    hit = torch.arange(int(off[-1]), device="cuda") - off[event] + b.hit_off[which[event]]
    x, y = b.x[hit].double(), b.y[hit].double()
    c, s = torch.cos(turn)[event], torch.sin(turn)[event]
    x, y = c * x - s * y, s * x + c * y
    z, plane = b.z[hit], b.plane[hit]
    planes = synth.WORKLOADS[case["workload"]].n_planes
    order = torch.argsort((event * planes + plane).double() * 8.0 + torch.atan2(y, x))
    return etx.Batch(n, int(off[-1]), off, x[order].float(), y[order].float(), z[order].contiguous(),
                     plane[order].contiguous())


def _weights(case):
    w = synth.WORKLOADS[case["workload"]]
    if case["weights"] == "trained":
        return synth.trained_weights(w)
    weights = synth.xavier_weights(w)
    if case["call"] == "train_gnn":      # the network trains on the rough graph of a trained embedding
        weights["emb"] = synth.trained_weights(w)["emb"]
    return weights


def _prefilter():
    (w1, b1), (w2, b2), (w3, b3) = [(0.02 * W, b.copy()) for W, b in synth.xavier_prefilter()]
    w1[:, 0], w2[:, 0], w2[0, :] = 0, 0, 0
    w1[5, 0], w2[0, 0], w3[0, 0], b3[0] = 1.0, 1.0, -SLOPE, SLOPE * CUT
    return np.concatenate([a.ravel() for a in (w1, b1, w2, b2, w3, b3)]).astype(np.float32)


def _capacity(case, n_hits):
    """Edge capacity: the k_max bound for dense graphs (None), eight candidates per hit for sparse ones."""
    return None if case["weights"] == "random" else 8 * n_hits + 1024


# ----------------------------------------------------------------------------
# what a program holds before the call
# ----------------------------------------------------------------------------

def prepare(case, seed):
    make = _prepare_run if case["call"] in ("run", "tracks") else _prepare_train
    state = make(case, int(seed))
    torch.cuda.synchronize()
    return state


def _prepare_run(case, seed):
    w = _workload(case)
    b = _batch(case, seed, _events(case, seed))
    p = etx.Pipeline(w, _weights(case), precision=PRECISION[case["precision"]])
    if case["compact"]:
        etx.etx_set_option(p.ctx, etx.ETX_OPT_COMPACT_STATE, 1)
    if case["precision"] in ("fp8", "int8"):
        calibration = etx.to_device(synth.generate_batch(w, 8, seed_space=99000))
        p.calibrate(calibration)
    if case["tuned"]:
        for key, value in (DENSE if case["weights"] == "random" else SPARSE).items():
            etx.etx_set_option(p.ctx, getattr(etx, "ETX_OPT_" + key), value)
    if case["prefilter"]:
        etx.etx_prefilter_set(p.ctx, _prefilter())
        etx.etx_prefilter_config(p.ctx, 1, TAU)
        etx.etx_prefilter_band(p.ctx, *BAND)
    etx.etx_set_option(p.ctx, etx.ETX_OPT_USE_GRAPH, int(case["graph"]))
    cap = _capacity(case, b.n_hits)
    state = dict(case=case, p=p, b=b, cap=cap, stream=torch.cuda.Stream() if case["graph"] else None)
    if case["call"] == "tracks":
        p.set_triplets(synth.trained_triplets(w))
        caps = state["caps"] = dict(triplet_capacity=8 * b.n_hits + 1024, track_capacity=b.n_hits + 1024,
                                    hit_capacity=4 * b.n_hits + 1024)
        p.allocate(b, cap, tri_caps=(caps["triplet_capacity"], caps["track_capacity"]))
        p.allocate_tracks(b, *caps.values())
        written = [p.tri_a, p.tri_b, p.tri_score, p.tri_kind, p.art_off, p.elb_off, p.event_track_off, p.track_off,
                   p.track_hits]
    else:
        p.allocate(b, cap)
        written = []
    # outputs are written up to the number of edges, triplets and tracks found
    for t in written + [p.src, p.dst, p.score, p.edge_off, p.labels]:
        t.zero_()
    return state


def _prepare_train(case, seed):
    w = _workload(case)
    host = _events(case, seed)
    b = etx.to_device(host)
    weights = _weights(case)
    state = dict(case=case, b=b, w=w, step=STEP, host=host)
    if case["call"] == "train_prefilter":
        p = etx.Pipeline(w, weights)
        n = etx.ETX_PF_NPARAM
        etx.etx_prefilter_set(p.ctx, _prefilter())
        labels, _ = prefilter_train.labels_from_full_pipeline(p, b, w.threshold)
        adam = etx.etx_prefilter_state(p.ctx)
        adam[2 * n:] = MOMENT2
        etx.etx_prefilter_state(p.ctx, adam)
        return dict(state, p=p, labels=labels)
    t = training.Trainer(w, weights)
    n = t.n_params
    etx.etx_train_params(t.ctx, np.concatenate([t.params(), np.zeros(n, np.float32), np.full(n, MOMENT2, np.float32)]))
    if case["call"] == "train_triplets":
        t.set_triplets(synth.xavier_triplets(w))
        n3 = etx.ETX_TRIPLET_NPARAM(w.gnn_hidden)
        head = etx.etx_train_triplet_params(t.ctx, n=n3)
        etx.etx_train_triplet_params(t.ctx, np.concatenate([head, np.zeros(n3, np.float32),
                                                            np.full(n3, MOMENT2, np.float32)]))
    truth, keep = training.truth_to_device(training.truth_arrays(host, w, np.random.default_rng(seed)))
    t.allocate_train(b)
    n_emb = sum(W.size + v.size for W, v in weights["emb"])
    return dict(state, p=t, truth=truth, keep=keep, n_emb=n_emb)


# ----------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------

def run(state):
    case, p, b = state["case"], state["p"], state["b"]
    call = case["call"]
    if call == "run":
        s = state["stream"]
        p.run(b, state["cap"], stream=s)
        if s is not None:
            torch.cuda.current_stream().wait_stream(s)
        return dict(src=p.src, dst=p.dst, score=p.score, edge_off=p.edge_off, labels=p.labels, status=p.status)
    if call == "tracks":
        p.run_tracks(b, edge_capacity=state["cap"], **state["caps"])
        return dict(src=p.src, dst=p.dst, score=p.score, edge_off=p.edge_off, labels=p.labels, status=p.status,
                    tri_a=p.tri_a, tri_b=p.tri_b, tri_score=p.tri_score, tri_kind=p.tri_kind, art_off=p.art_off,
                    elb_off=p.elb_off, event_track_off=p.event_track_off, track_off=p.track_off,
                    track_hits=p.track_hits, track_status=p.tstatus)
    state["step"] += 1
    lr, step, w = LR[call], state["step"], state["w"]
    if call == "train_prefilter":
        loss = p.prefilter_train_step(b, state["labels"], lr, POS_WEIGHT, step)
        return dict(loss=loss, grad=p.view(b, etx.ETX_VIEW_PF_GRAD, torch.float32)[:etx.ETX_PF_NPARAM])
    if call == "train_embed":
        margin, r_train = _margin(w)
        loss = p.embed_step(b, state["truth"], margin, W_GEN, r_train, lr, step)
        return dict(loss=loss, grad=p.train_view(b, 0, torch.float32)[:state["n_emb"]])
    if call == "train_gnn":
        loss = p.gnn_step(b, state["truth"], ALPHA, GAMMA, lr, step)
        return dict(loss=loss, grad=p.train_view(b, 0, torch.float32)[state["n_emb"]:])
    loss = p.triplet_step(b, state["truth"], ALPHA, GAMMA, lr, step)
    return dict(loss=loss, grad=p.train_view(b, 0, torch.float32)[state["n_emb"]:],
                grad_triplets=p.triplet_view(b, 0, torch.float32))


def _margin(w):
    margin = w.radius ** 2 / 0.9
    return margin, float(np.sqrt(1.5 * margin))


# ----------------------------------------------------------------------------
# the work a pass cannot do without
# ----------------------------------------------------------------------------

def work(case):
    wl = synth.WORKLOADS[case["workload"]]
    name = case["workload"]
    n = case["events"] * (case["tracks"] * HITS_PER_TRACK[name] if case["tracks"] else HITS[name])
    sparse = case["weights"] == "trained" or case["call"] == "train_gnn"
    edges = n * EDGES[name][1 if sparse else 0]
    H, S, W, L, D = wl.gnn_hidden, wl.gnn_steps, wl.emb_hidden, wl.emb_layers, wl.emb_dim
    embed = n * 2 * (3 * W + (L - 1) * W * W + W * D)
    gnn_edges = edges * (0.67 if case.get("prefilter") else 1.0)
    # layer 1 of the edge networks split by input block: the node blocks once per hit
    network = n * 2 * (3 * H + H * H + 2 * H * H) + gnn_edges * 2 * H * H \
        + S * (n * 2 * (4 * H * H + 2 * H * H) + gnn_edges * 4 * H * H) + gnn_edges * (2 * H * H + 2 * H)
    pairs = edges * 2 * D
    mlp = edges * 2 * (6 * 32 + 32 * 32 + 32)
    hits_in, edges_out = 20 * n, 12 * gnn_edges
    call = case["call"]
    if call == "run":
        return dict(bytes=hits_in + edges_out + 4 * n, flops=embed + pairs + network + (mlp if case["prefilter"] else 0))
    if call == "tracks":
        triplets = 0.8 * n
        return dict(bytes=hits_in + edges_out + 4 * n + 13 * triplets + 5 * n,
                    flops=embed + pairs + network + triplets * 2 * (3 * H * H + H))
    # a training step: forward, and twice that backward (inputs and weights); parameters and moments read and written
    params = 3 * W + (L - 1) * W * W + W * D if call == "train_embed" else S * 8 * H * H + 6 * H * H
    state = 24 * params
    if call == "train_prefilter":
        return dict(bytes=hits_in + edges, flops=embed + pairs + 3 * mlp)
    if call == "train_embed":
        return dict(bytes=hits_in + 24 * n + state, flops=3 * embed + pairs)
    triplets = 0.8 * n * 2 * (3 * H * H + H) if call == "train_triplets" else 0
    return dict(bytes=hits_in + 24 * n + state, flops=embed + pairs + 3 * (network + triplets))


# ----------------------------------------------------------------------------
# the same in 64 bits, in plain torch
# ----------------------------------------------------------------------------

# Two hits whose distance lies this near the radius, or two candidates of a full row this near in distance, may
# fall on either side in single precision: the graph, and with it every output, then has no single 64-bit value.
_DOUBT = 3e-7
_MOST_HITS = 40000


class _Doubt(Exception):
    pass


def exact(case, seed):
    if case["call"] in ("tracks", "train_prefilter") or case.get("precision", "fp32") != "fp32" or case.get("prefilter"):
        return None
    if case["events"] > _BASE or case["events"] * HITS[case["workload"]] > _MOST_HITS:
        return None
    host = _events(case, int(seed))
    try:
        if case["call"] == "run":
            return _exact_run(case, host)
        return _exact_train(case, host, int(seed))
    except _Doubt:
        return None


def _inputs64(host, w):
    x, y, z = (torch.as_tensor(host[k], device="cuda").double() for k in ("x", "y", "z"))
    cyl = torch.stack([torch.sqrt(x * x + y * y) / w.r_scale, torch.atan2(y, x) / math.pi, z / w.z_scale], 1)
    return cyl, torch.stack([x / w.r_scale, y / w.r_scale, z / w.z_scale], 1)


def _weights64(weights, grad=False):
    t = lambda a: torch.as_tensor(a, device="cuda").double().requires_grad_(grad)
    return {k: [(t(W), t(b)) for W, b in v] for k, v in weights.items()}


def _embed64(cyl, layers):
    for i, (W, b) in enumerate(layers):
        cyl = cyl @ W + b
        if i + 1 < len(layers):
            cyl = torch.relu(cyl)
    return cyl


def _radius64(host, emb, w, radius):
    """The edges (src, dst), source-major, of every event."""
    r = float(np.float32(radius))
    plane = torch.as_tensor(host["plane"], device="cuda").long()
    src, dst = [], []
    for a, b in zip(host["hit_off"][:-1], host["hit_off"][1:]):
        e, p = emb[a:b], plane[a:b]
        for k in range(w.n_planes - 1):
            s = torch.nonzero(p == k).flatten()
            t = torch.nonzero((p > k) & (p <= k + w.plane_window)).flatten()
            if not len(s) or not len(t):
                continue
            d = torch.sqrt(((e[s][:, None] - e[t][None]) ** 2).sum(2))
            if bool(((d - r).abs() < _DOUBT).any()):
                raise _Doubt
            near = d < r
            full = near.sum(1) > w.k_max
            if bool(full.any()):
                v = torch.sort(d[full], 1).values
                if bool((v[:, w.k_max] - v[:, w.k_max - 1] < _DOUBT).any()):
                    raise _Doubt
                last = torch.full_like(d[:, 0], math.inf)
                last[full] = v[:, w.k_max - 1]
                near &= d <= last[:, None]
            i, j = torch.nonzero(near, as_tuple=True)
            src.append(s[i] + a)
            dst.append(t[j] + a)
    none = torch.zeros(0, dtype=torch.int64, device="cuda")
    src, dst = torch.cat(src + [none]), torch.cat(dst + [none])
    order = torch.argsort(src * (int(host["hit_off"][-1]) + 1) + dst)
    return src[order], dst[order]


def _block64(x, layer):
    y = x @ layer[0] + layer[1]
    y = y - y.mean(1, keepdim=True)
    return torch.relu(y / torch.sqrt((y * y).mean(1, keepdim=True) + 1e-5))


def _network64(cart, src, dst, weights, steps):
    mlp = lambda x, net: _block64(_block64(x, weights[net][0]), weights[net][1])
    h = mlp(cart, "node_enc")
    e = mlp(torch.cat([h[src], h[dst]], 1), "edge_enc")
    for k in range(steps):
        out = torch.zeros_like(h).index_add(0, src, e)
        inn = torch.zeros_like(h).index_add(0, dst, e)
        h = h + mlp(torch.cat([h, out, inn], 1), f"node{k}")
        e = e + mlp(torch.cat([e, h[src], h[dst]], 1), f"edge{k}")
    (W, b), = weights["cls"][1:]
    return (_block64(e, weights["cls"][0]) @ W + b).flatten(), e


def _exact_run(case, host):
    w = _workload(case)
    weights = _weights64(_weights(case))
    cyl, cart = _inputs64(host, w)
    src, dst = _radius64(host, _embed64(cyl, weights["emb"]), w, w.radius)
    logit, _ = _network64(cart, src, dst, weights, w.gnn_steps)
    cap = _capacity(case, len(cyl))
    score = torch.zeros(len(cyl) * w.k_max if cap is None else cap, dtype=torch.float64, device="cuda")
    score[:len(logit)] = torch.sigmoid(logit)
    return dict(src=None, dst=None, score=score, edge_off=None, labels=None, status=None)


def _focal64(logit, label):
    """Mean sigmoid focal loss."""
    if not len(logit):
        return logit.sum()
    p = torch.sigmoid(logit)
    y = label.double()
    right = p * y + (1 - p) * (1 - y)
    ce = torch.nn.functional.binary_cross_entropy_with_logits(logit, y, reduction="none")
    return ((ALPHA * y + (1 - ALPHA) * (1 - y)) * (1 - right) ** GAMMA * ce).mean()


def _exact_train(case, host, seed):
    w = _workload(case)
    weights = _weights64(_weights(case), grad=True)
    cyl, cart = _inputs64(host, w)
    truth = {k: torch.as_tensor(v, device="cuda") for k, v in
             training.truth_arrays(host, w, np.random.default_rng(seed)).items()}
    succ = truth["succ"].long()
    emb = _embed64(cyl, weights["emb"])
    if case["call"] == "train_embed":
        margin, r_train = _margin(w)
        src, dst = _radius64(host, emb.detach(), w, r_train)
        query = truth["query"].bool()
        rnd = truth["rnd"].long()
        q = torch.nonzero(query & (succ >= 0)).flatten()
        hard = query[src] & (truth["particle"][dst] >= 0) & (dst != succ[src])
        r = torch.nonzero(query & (rnd >= 0) & (rnd != succ)).flatten()
        fs, fd = torch.cat([src[hard], r]), torch.cat([dst[hard], rnd[r]])
        margin = float(np.float32(margin))
        d2 = ((emb[fs] - emb[fd]) ** 2).sum(1)
        if bool(((d2 - margin).abs() < _DOUBT * 0.1).any()):
            raise _Doubt
        loss = torch.relu(margin - d2).mean() + W_GEN * ((emb[q] - emb[succ[q]]) ** 2).sum(1).mean()
        loss.backward()
        return dict(loss=loss.detach().reshape(1), grad=_flat_grad(weights, ["emb"]))
    src, dst = _radius64(host, emb.detach(), w, w.radius)
    logit, e = _network64(cart, src, dst, weights, w.gnn_steps)
    label = dst == succ[src]
    if case["call"] == "train_triplets":
        label = label | (dst == truth["succ2"].long()[src])
    losses = [_focal64(logit, label)]
    nets = [k for k, _ in training.weight_order(w) if k != "emb"]
    if case["call"] == "train_gnn":
        losses[0].backward()
        return dict(loss=losses[0].detach().reshape(1), grad=_flat_grad(weights, nets))
    score = torch.sigmoid(logit.detach())
    if bool(((score - 0.5).abs() < 1e-5).any()):
        raise _Doubt
    heads = _weights64(synth.xavier_triplets(w), grad=True)
    for head, (a, b, y) in _triplets64(host, src, dst, score >= 0.5, truth).items():
        x = torch.cat([e[a], e[b]], 1)
        x = _block64(_block64(x, heads[head][0]), heads[head][1])
        losses.append(_focal64((x @ heads[head][2][0] + heads[head][2][1]).flatten(), y))
    sum(losses).backward()
    return dict(loss=torch.stack(losses).detach(), grad=_flat_grad(weights, nets),
                grad_triplets=_flat_grad(heads, ["art", "elb"]))


def _triplets64(host, src, dst, keep, truth):
    """Articulations and elbows of the kept graph, each as (first edges, second edges, labels)."""
    plane, p1, p2, s1, s2 = (np.asarray(a) for a in (host["plane"], *(truth[k].cpu().numpy() for k in (
        "particle", "particle2", "succ", "succ2"))))
    ids = torch.nonzero(keep).flatten().cpu().numpy()
    es, ed = src.cpu().numpy(), dst.cpu().numpy()
    out, inn = {}, {}
    for i in ids:
        out.setdefault(es[i], []).append(i)
        inn.setdefault(ed[i], []).append(i)
    owners = lambda h: {p for p in (p1[h], p2[h]) if p >= 0}

    def follows(q, a, b):       # b is particle q's next hit after a
        return (p1[a] == q and s1[a] == b) or (p2[a] == q and s2[a] == b)

    art, elb = [], []
    for i in ids:
        for j in out.get(ed[i], []):
            a, c, b = es[i], ed[i], ed[j]
            art.append((i, j, any(follows(q, a, c) and follows(q, c, b) for q in owners(a) & owners(c))))
    for side, far, near in ((out, ed, es), (inn, es, ed)):
        for c, row in side.items():
            for x in range(len(row)):
                for y in range(x + 1, len(row)):
                    i, j = row[x], row[y]
                    if abs(int(plane[far[j]]) - int(plane[c])) < abs(int(plane[far[i]]) - int(plane[c])):
                        i, j = j, i
                    elb.append((i, j, bool(owners(far[i]) & owners(far[j]) & owners(c))))
    t = lambda v, dt: torch.as_tensor(np.array(v), dtype=dt, device="cuda")
    return {k: tuple(t([r[c] for r in v], torch.bool if c == 2 else torch.int64) for c in range(3))
            for k, v in (("art", art), ("elb", elb))}


def _flat_grad(weights, nets):
    return torch.cat([(torch.zeros_like(p) if p.grad is None else p.grad).reshape(-1)
                      for k in nets for layer in weights[k] for p in layer])
