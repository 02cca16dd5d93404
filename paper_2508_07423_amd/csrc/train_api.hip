// Host side of in-library training: the training parameters in the context,
// the workspace layout of a training step, and the step sequences.
//
// The graph of a step is built by the inference stages (bucketing, radius
// graph, CSC permutation); the embedding step builds it in its own training
// embedding at the training radius (hard negatives, thesis ch. 8), the
// network step with the context's inference embedding (the rough graph).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <initializer_list>
#include <vector>

#include "internal.hpp"
#include "train.hpp"

namespace etx {

size_t blob_floats_of(const etx_config& c);
etx_status check_run(const etx_ctx* ctx, const etx_hits* hits, const etx_out* out, void* ws, size_t ws_bytes,
                     WsLayout* L);
etx_status rebuild_weights(etx_ctx* ctx, const float* payload);

namespace {

size_t a256(size_t x) { return (x + 255) & ~size_t(255); }

// Most partials of any number of rows up to `rows`.
size_t most_chunks(int64_t rows) { return (size_t)std::min<int64_t>(rows, kTrainChunks); }

// offsets (floats) of the parameter blocks in the blob payload
struct ParamMap {
  int64_t emb[8];           // embedding layer l
  int64_t ne1, ne2, ee1, ee2, nn1[16], nn2[16], en1[16], en2[16], cls1, cls2, gnn_begin, total;
};

ParamMap param_map(const etx_config& c) {
  ParamMap P{};
  int64_t o = 0;
  const int64_t W = c.emb_hidden, D = c.emb_dim, H = c.gnn_hidden;
  for (int l = 0; l <= c.emb_layers && l < 8; ++l) {
    const int64_t K = l == 0 ? 3 : W, M = l < c.emb_layers ? W : D;
    P.emb[l] = o;
    o += K * M + M;
  }
  P.gnn_begin = o;
  auto take = [&](int64_t K, int64_t M) {
    int64_t at = o;
    o += K * M + M;
    return at;
  };
  P.ne1 = take(3, H);
  P.ne2 = take(H, H);
  P.ee1 = take(2 * H, H);
  P.ee2 = take(H, H);
  for (int k = 0; k < c.gnn_steps; ++k) {
    P.nn1[k] = take(3 * H, H);
    P.nn2[k] = take(H, H);
    P.en1[k] = take(3 * H, H);
    P.en2[k] = take(H, H);
  }
  P.cls1 = take(H, H);
  P.cls2 = take(H, 1);
  P.total = o;
  return P;
}

struct TrainLayout {
  // embedding
  size_t emb_z[4], de, g_gen, g_rnd, g_edge, counts;
  // network
  size_t hst, mo, mi, yh_n, rs_n, est, yh_e, rs_e, lab, de_e, dxs, dxd, dh, dmo, dmi;
  // shared
  size_t part, grad, lpart, loss;
  size_t total;
};

TrainLayout train_layout(const etx_ctx* ctx, const WsLayout& L, int64_t n, int64_t E) {
  const etx_config& c = ctx->cfg;
  const int64_t H = c.gnn_hidden, S = c.gnn_steps, W = c.emb_hidden, D = c.emb_dim;
  TrainLayout T{};
  size_t o = L.total;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o += a256(std::max<size_t>(bytes, 1));
    return at;
  };
  const size_t f = sizeof(float);
  for (int l = 0; l < c.emb_layers; ++l) T.emb_z[l] = take(f * n * W);
  T.de = take(f * n * kDpad);
  T.g_gen = take(f * n * D);
  T.g_rnd = take(f * n * D);
  T.g_edge = take(f * E * D);
  T.counts = take(f * 2 * kHingeBlocks);
  T.hst = take(f * (S + 1) * n * H);
  T.mo = take(f * S * n * H);
  T.mi = take(f * S * n * H);
  T.yh_n = take(f * (2 + 2 * S) * n * H);
  T.rs_n = take(f * (2 + 2 * S) * n);
  T.est = take(f * (S + 1) * E * H);
  T.yh_e = take(f * (2 + 2 * S) * E * H);
  T.rs_e = take(f * (2 + 2 * S) * E);
  T.lab = take(E);
  T.de_e = take(f * E * H);
  T.dxs = take(f * E * H);
  T.dxd = take(f * E * H);
  T.dh = take(f * n * H);
  T.dmo = take(f * n * H);
  T.dmi = take(f * n * H);
  // gradient partials: the embedding's over hits, the network's over hits and edges (at most one per pair of hits)
  const ParamMap P = param_map(c);
  const int64_t some = std::min<int64_t>(n, kTrainChunks);
  T.part = take(f * most_chunks(std::max(some, std::min(E, some * (some - 1) / 2))) *
                std::max(P.gnn_begin, P.total - P.gnn_begin));
  T.grad = take(f * P.total);
  T.lpart = take(f * std::max(3 * kTrainChunks, kHingeBlocks));
  T.loss = take(f * 4);
  T.total = o;
  return T;
}

// The triplet part of a network step's workspace (after the TrainLayout).
struct TripLayout {
  size_t ta, tb, kind, tscore, art_off, elb_off, tstatus, tri, lab, dxa, dxb, part, tgrad, total;
  TriLayout TL;
};

TripLayout trip_layout(const etx_ctx* ctx, size_t base, int64_t n_events, int64_t n, int64_t E, int64_t tcap) {
  const int64_t H = ctx->cfg.gnn_hidden;
  TripLayout X{};
  size_t o = base;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o += a256(std::max<size_t>(bytes, 1));
    return at;
  };
  const size_t f = sizeof(float), T = (size_t)tcap;
  X.ta = take(4 * T);
  X.tb = take(4 * T);
  X.kind = take(T);
  X.tscore = take(f * T);
  X.art_off = take(8 * (size_t)(n_events + 1));
  X.elb_off = take(8 * (size_t)(n_events + 1));
  X.tstatus = take(8 * 4);
  X.TL = tri_layout(n_events, n, E, tcap, 0);
  X.tri = take(X.TL.total);
  X.lab = take(T);
  X.dxa = take(f * T * H);
  X.dxb = take(f * T * H);
  X.part = take(f * ETX_TRIPLET_NPARAM(H) * most_chunks(tcap));
  X.tgrad = take(f * ETX_TRIPLET_NPARAM(H));
  X.total = o;
  return X;
}

}  // namespace
}  // namespace etx

using namespace etx;

#define F(off) reinterpret_cast<float*>(ws + (off))
#define HIPCHK(x)                              \
  do {                                         \
    hipError_t e_ = (x);                       \
    if (e_ != hipSuccess) {                    \
      note_error(what, e_);                    \
      return ETX_ERR_HIP;                      \
    }                                          \
  } while (0)

namespace etx {
void note_error(const char* what, hipError_t e);
}

extern "C" {

etx_status etx_train_begin(etx_ctx* ctx) {
  if (!ctx) return ETX_ERR_INVALID_ARG;
  const char* what = "etx_train_begin";
  if (hipSetDevice(ctx->device) != hipSuccess) return ETX_ERR_HIP;
  const size_t n = blob_floats_of(ctx->cfg);
  if (!ctx->dev_train) HIPCHK(hipMalloc(&ctx->dev_train, sizeof(float) * 3 * n));
  HIPCHK(hipMemcpy(ctx->dev_train, ctx->blob.data() + 32, sizeof(float) * n, hipMemcpyHostToDevice));
  HIPCHK(hipMemset(ctx->dev_train + n, 0, sizeof(float) * 2 * n));
  ctx->tri_train_fresh = true;
  return ETX_OK;
}

}  // extern "C"

namespace {

// the triplet classifiers' training state, (re)started from the context's
// triplet parameters after etx_train_begin
etx_status tri_train_state(etx_ctx* ctx) {
  const char* what = "triplet training state";
  if (!ctx->dev_train || ctx->tri_host.empty()) return ETX_ERR_INVALID_ARG;
  const size_t np = ctx->tri_host.size();
  if (!ctx->dev_tri_train) HIPCHK(hipMalloc(&ctx->dev_tri_train, sizeof(float) * 3 * np));
  if (ctx->tri_train_fresh) {
    HIPCHK(hipMemcpy(ctx->dev_tri_train, ctx->tri_host.data(), sizeof(float) * np, hipMemcpyHostToDevice));
    HIPCHK(hipMemset(ctx->dev_tri_train + np, 0, sizeof(float) * 2 * np));
    ctx->tri_train_fresh = false;
  }
  return ETX_OK;
}

}  // namespace

extern "C" {

etx_status etx_train_triplet_params(etx_ctx* ctx, float* host, int64_t n, int32_t set) {
  if (!ctx || !host || (set != 0 && set != 1)) return ETX_ERR_INVALID_ARG;
  if (hipSetDevice(ctx->device) != hipSuccess) return ETX_ERR_HIP;
  etx_status st = tri_train_state(ctx);
  if (st != ETX_OK) return st;
  const int64_t np = (int64_t)ctx->tri_host.size();
  if (n < 1 || n > 3 * np) return ETX_ERR_INVALID_ARG;
  const char* what = "etx_train_triplet_params";
  HIPCHK(set ? hipMemcpy(ctx->dev_tri_train, host, sizeof(float) * n, hipMemcpyHostToDevice)
             : hipMemcpy(host, ctx->dev_tri_train, sizeof(float) * n, hipMemcpyDeviceToHost));
  return ETX_OK;
}

etx_status etx_train_params(etx_ctx* ctx, float* host, int64_t n, int32_t set) {
  if (!ctx || !host || !ctx->dev_train) return ETX_ERR_INVALID_ARG;
  const int64_t nb = (int64_t)blob_floats_of(ctx->cfg);
  if (n < 1 || n > 3 * nb) return ETX_ERR_INVALID_ARG;
  const char* what = "etx_train_params";
  if (hipSetDevice(ctx->device) != hipSuccess) return ETX_ERR_HIP;
  HIPCHK(set ? hipMemcpy(ctx->dev_train, host, sizeof(float) * n, hipMemcpyHostToDevice)
             : hipMemcpy(host, ctx->dev_train, sizeof(float) * n, hipMemcpyDeviceToHost));
  return ETX_OK;
}

etx_status etx_train_apply(etx_ctx* ctx) {
  if (!ctx || !ctx->dev_train) return ETX_ERR_INVALID_ARG;
  const char* what = "etx_train_apply";
  if (hipSetDevice(ctx->device) != hipSuccess) return ETX_ERR_HIP;
  std::vector<float> p(blob_floats_of(ctx->cfg));
  HIPCHK(hipMemcpy(p.data(), ctx->dev_train, sizeof(float) * p.size(), hipMemcpyDeviceToHost));
  etx_status st = rebuild_weights(ctx, p.data());
  if (st != ETX_OK || !ctx->dev_tri_train || ctx->tri_train_fresh) return st;
  std::vector<float> q(ctx->tri_host.size());
  HIPCHK(hipMemcpy(q.data(), ctx->dev_tri_train, sizeof(float) * q.size(), hipMemcpyDeviceToHost));
  return etx_triplet_set(ctx, q.data(), (int64_t)q.size());
}

etx_status etx_train_workspace_size(const etx_ctx* ctx, int64_t n_events, int64_t n_hits, int64_t edge_capacity,
                                    size_t* bytes) {
  if (!ctx || !bytes || n_events < 0 || n_hits < 0 || edge_capacity < 0) return ETX_ERR_INVALID_ARG;
  const WsLayout L = ws_layout(ctx, n_events, n_hits, edge_capacity);
  *bytes = train_layout(ctx, L, n_hits, edge_capacity).total;
  return ETX_OK;
}

etx_status etx_train_triplet_workspace_size(const etx_ctx* ctx, int64_t n_events, int64_t n_hits,
                                            int64_t edge_capacity, int64_t triplet_capacity, size_t* bytes) {
  if (!ctx || !bytes || n_events < 0 || n_hits < 0 || edge_capacity < 0 || triplet_capacity < 0)
    return ETX_ERR_INVALID_ARG;
  const WsLayout L = ws_layout(ctx, n_events, n_hits, edge_capacity);
  const TrainLayout T = train_layout(ctx, L, n_hits, edge_capacity);
  *bytes = trip_layout(ctx, T.total, n_events, n_hits, edge_capacity, triplet_capacity).total;
  return ETX_OK;
}

etx_status etx_train_triplet_view(const etx_ctx* ctx, int64_t n_events, int64_t n_hits, int64_t edge_capacity,
                                  int64_t triplet_capacity, int32_t which, size_t* offset, size_t* bytes) {
  if (!ctx || !offset || !bytes || triplet_capacity < 0) return ETX_ERR_INVALID_ARG;
  const WsLayout L = ws_layout(ctx, n_events, n_hits, edge_capacity);
  const TrainLayout T = train_layout(ctx, L, n_hits, edge_capacity);
  const TripLayout X = trip_layout(ctx, T.total, n_events, n_hits, edge_capacity, triplet_capacity);
  const size_t tc = (size_t)triplet_capacity;
  switch (which) {
    case 0: *offset = X.tgrad; *bytes = sizeof(float) * ETX_TRIPLET_NPARAM(ctx->cfg.gnn_hidden); break;
    case 1: *offset = X.lab; *bytes = tc; break;
    case 2: *offset = X.ta; *bytes = 4 * tc; break;
    case 3: *offset = X.tb; *bytes = 4 * tc; break;
    case 4: *offset = X.kind; *bytes = tc; break;
    case 5: *offset = X.art_off; *bytes = 8 * (size_t)(n_events + 1); break;
    case 6: *offset = X.elb_off; *bytes = 8 * (size_t)(n_events + 1); break;
    default: return ETX_ERR_INVALID_ARG;
  }
  return ETX_OK;
}

etx_status etx_train_view(const etx_ctx* ctx, int64_t n_events, int64_t n_hits, int64_t edge_capacity, int32_t which,
                          size_t* offset, size_t* bytes) {
  if (!ctx || !offset || !bytes) return ETX_ERR_INVALID_ARG;
  const WsLayout L = ws_layout(ctx, n_events, n_hits, edge_capacity);
  const TrainLayout T = train_layout(ctx, L, n_hits, edge_capacity);
  switch (which) {
    case 0: *offset = T.grad; *bytes = sizeof(float) * blob_floats_of(ctx->cfg); break;
    case 1: *offset = T.loss; *bytes = sizeof(float) * 4; break;
    case 2: *offset = T.lab; *bytes = edge_capacity; break;
    default: return ETX_ERR_INVALID_ARG;
  }
  return ETX_OK;
}

}  // extern "C"

namespace {

// the inference stages that build a batch's graph: bucketing, (embedding), radius graph, CSC permutation
hipError_t build_graph(const RunArgs& a, bool inference_embedding) {
  hipError_t e;
  if ((e = launch_init_status(a)) != hipSuccess) return e;
  if ((e = launch_validate(a)) != hipSuccess) return e;
  if ((e = launch_bucket(a)) != hipSuccess) return e;
  if (inference_embedding && (e = launch_embed(a)) != hipSuccess) return e;
  return hipSuccess;
}

hipError_t radius_and_csc(const RunArgs& a) {
  hipError_t e;
  if (a.ctx->radius_single) {
    if ((e = launch_radius(a, 2, false)) != hipSuccess) return e;
    if ((e = launch_scan_counts(a, false)) != hipSuccess) return e;
    if ((e = launch_slots_copy(a, false)) != hipSuccess) return e;
  } else {
    if ((e = launch_radius(a, 0, false)) != hipSuccess) return e;
    if ((e = launch_scan_counts(a, false)) != hipSuccess) return e;
    if ((e = launch_radius(a, 1, false)) != hipSuccess) return e;
  }
  return launch_csc(a);
}

}  // namespace

extern "C" {

etx_status etx_train_embed_step(etx_ctx* ctx, const etx_hits* hits, etx_out* out, const etx_truth* truth,
                                float margin, float w_gen, float r_train, float lr, int64_t step, float* loss_dev,
                                void* ws_, size_t ws_bytes, etx_stream stream) {
  const char* what = "etx_train_embed_step";
  if (!ctx || !hits || !out || !truth || !ctx->dev_train) return ETX_ERR_INVALID_ARG;
  if (!truth->particle || !truth->succ || !truth->pred || !truth->query || !truth->rnd || !truth->rnd_ptr ||
      (!truth->rnd_src && hits->n_hits > 0))
    return ETX_ERR_INVALID_ARG;
  if (!(margin > 0) || !(w_gen > 0) || !(r_train > 0) || !(lr >= 0) || step < 1) return ETX_ERR_INVALID_ARG;
  const etx_config& c = ctx->cfg;
  if (c.emb_dim != 4 && c.emb_dim != 8 && c.emb_dim != 12 && c.emb_dim != 16) return ETX_ERR_UNSUPPORTED;
  WsLayout L;
  etx_status st = check_run(ctx, hits, out, ws_, ws_bytes, &L);
  if (st != ETX_OK) return st;
  const int64_t n = hits->n_hits, cap = out->edge_capacity;
  const TrainLayout T = train_layout(ctx, L, n, cap);
  if (ws_bytes < T.total) return ETX_ERR_INVALID_ARG;
  if (hipSetDevice(ctx->device) != hipSuccess) return ETX_ERR_HIP;
  char* ws = static_cast<char*>(ws_);
  hipStream_t s = static_cast<hipStream_t>(stream);
  RunArgs a{ctx, *hits, *out, L, ws, s, false, ETX_FP32};
  const ParamMap P = param_map(c);
  float* prm = ctx->dev_train;
  float* grad = F(T.grad);
  const int64_t* status = out->status;
  const int W = c.emb_hidden, D = c.emb_dim;
  HIPCHK(build_graph(a, false));
  // training embedding: forward, keeping every hidden layer's z; the output goes to the embedding buffer
  const int NL = c.emb_layers;
  EmbTrain Em{};
  Em.n = n;
  Em.x = hits->x;
  Em.y = hits->y;
  Em.z = hits->z;
  Em.inv_r = 1.0f / c.r_scale_mm;
  Em.inv_z = 1.0f / c.z_scale_mm;
  for (int l = 0; l <= NL; ++l) {
    Em.W[l] = prm + P.emb[l];
    Em.o[l] = P.emb[l];
    if (l < NL) Em.zs[l] = F(T.emb_z[l]);
  }
  Em.emb = F(L.emb);
  Em.de = F(T.de);
  Em.D = D;
  Em.part = F(T.part);
  Em.part_stride = P.gnn_begin;
  Em.status = status;
  HIPCHK(launch_emb_fwd(Em, W, NL, ctx, s));
  // hard negatives: the radius graph of the training embedding at the training radius
  RunArgs ar = a;
  ar.radius_override = r_train;
  HIPCHK(radius_and_csc(ar));
  HingeArgs Hg{};
  Hg.n = n;
  Hg.emb = F(L.emb);
  Hg.lde = kDpad;
  Hg.query = truth->query;
  Hg.succ = truth->succ;
  Hg.pred = truth->pred;
  Hg.particle = truth->particle;
  Hg.rnd = truth->rnd;
  Hg.rnd_ptr = truth->rnd_ptr;
  Hg.rnd_src = truth->rnd_src;
  Hg.row_ptr = reinterpret_cast<const int64_t*>(ws + L.row_ptr);
  Hg.dst = out->dst;
  Hg.col_ptr = reinterpret_cast<const int64_t*>(ws + L.col_ptr);
  Hg.csc = reinterpret_cast<const int32_t*>(ws + L.csc);
  Hg.margin = margin;
  Hg.w_gen = w_gen;
  Hg.count_part = F(T.counts);
  Hg.loss_part = F(T.lpart);
  Hg.g_gen = F(T.g_gen);
  Hg.g_rnd = F(T.g_rnd);
  Hg.g_edge = F(T.g_edge);
  Hg.de = F(T.de);
  Hg.ldde = kDpad;
  Hg.status = status;
  HIPCHK(launch_hinge(Hg, D, s));
  HIPCHK(launch_emb_bwd(Em, W, NL, s));
  const int64_t nb = (int64_t)blob_floats_of(c);
  GradAdam G{};
  G.set[0].part = F(T.part);
  G.set[0].stride = P.gnn_begin;
  G.set[0].n = G.set[0].b0 = P.gnn_begin;
  G.set[0].g0 = net_groups(n);
  G.set[0].grad = grad;
  G.set[0].p = prm;
  G.set[0].m = prm + nb;
  G.set[0].v = prm + 2 * nb;
  G.lr = lr;
  G.loss_part[0] = F(T.lpart);
  G.loss_n[0] = hinge_blocks(n);
  G.loss = F(T.loss);
  G.loss_dev = loss_dev;
  G.status = status;
  HIPCHK(launch_grad_adam(G, step, s));
  return ETX_OK;
}

}  // extern "C"

namespace {

// One network step; tcap >= 0 adds the triplet term of eq. gnn-loss.
etx_status gnn_step(etx_ctx* ctx, const etx_hits* hits, etx_out* out, const etx_truth* truth, float alpha,
                    float gamma, float lr, int64_t step, int64_t tcap, int64_t* needed, float* loss_dev, void* ws_,
                    size_t ws_bytes, etx_stream stream) {
  const char* what = tcap >= 0 ? "etx_train_triplet_step" : "etx_train_gnn_step";
  if (!ctx || !hits || !out || !truth || !truth->succ || !ctx->dev_train) return ETX_ERR_INVALID_ARG;
  if (!(alpha >= 0 && alpha <= 1) || !(gamma >= 0) || !(lr >= 0) || step < 1) return ETX_ERR_INVALID_ARG;
  const bool trip = tcap >= 0;
  if (trip && (!truth->particle || tcap >= 0x7fffffffLL)) return ETX_ERR_INVALID_ARG;
  const etx_config& c = ctx->cfg;
  WsLayout L;
  etx_status st = check_run(ctx, hits, out, ws_, ws_bytes, &L);
  if (st != ETX_OK) return st;
  const int64_t n = hits->n_hits, cap = out->edge_capacity;
  const TrainLayout T = train_layout(ctx, L, n, cap);
  if (ws_bytes < T.total) return ETX_ERR_INVALID_ARG;
  TripLayout X{};
  if (trip) {
    X = trip_layout(ctx, T.total, hits->n_events, n, cap, tcap);
    if (ws_bytes < X.total) return ETX_ERR_INVALID_ARG;
    if (hipSetDevice(ctx->device) != hipSuccess) return ETX_ERR_HIP;
    if ((st = tri_train_state(ctx)) != ETX_OK) return st;
  }
  if (hipSetDevice(ctx->device) != hipSuccess) return ETX_ERR_HIP;
  char* ws = static_cast<char*>(ws_);
  hipStream_t s = static_cast<hipStream_t>(stream);
  RunArgs a{ctx, *hits, *out, L, ws, s, false, ETX_FP32};
  const ParamMap P = param_map(c);
  float* prm = ctx->dev_train;
  float* grad = F(T.grad);
  const int64_t* status = out->status;
  const int H = c.gnn_hidden, S = c.gnn_steps;
  HIPCHK(build_graph(a, true));
  HIPCHK(radius_and_csc(a));
  // the number of edges (this step synchronises the stream once)
  int64_t dev_status[2];
  int64_t E = 0;
  HIPCHK(hipMemcpyAsync(&E, ws + L.row_ptr + sizeof(int64_t) * n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  HIPCHK(hipMemcpyAsync(dev_status, out->status, sizeof(dev_status), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  if (dev_status[0] != ETX_OK) return static_cast<etx_status>(dev_status[0]);
  const int64_t nH = n * H, eH = E * H;
  auto hst = [&](int k) { return F(T.hst) + k * nH; };
  auto est = [&](int k) { return F(T.est) + k * eH; };
  // layers j of node rows: 0 ne1, 1 ne2, 2 + 2k nn1_k, 3 + 2k nn2_k; of edge rows: 0 ee1, 1 ee2, 2 + 2k en1_k, 3 + 2k en2_k
  NetStep base{};
  base.n = n;
  base.E = E;
  base.x = hits->x;
  base.y = hits->y;
  base.z = hits->z;
  base.inv_r = 1.0f / c.r_scale_mm;
  base.inv_z = 1.0f / c.z_scale_mm;
  base.row_ptr = reinterpret_cast<const int64_t*>(ws + L.row_ptr);
  base.col_ptr = reinterpret_cast<const int64_t*>(ws + L.col_ptr);
  base.csc = reinterpret_cast<const int32_t*>(ws + L.csc);
  base.src = out->src;
  base.dst = out->dst;
  base.lab = reinterpret_cast<uint8_t*>(ws + T.lab);
  base.succ = truth->succ;
  base.succ2 = truth->succ2;
  base.alpha = alpha;
  base.gamma = gamma;
  base.lpart = F(T.lpart);
  base.score = trip ? out->score : nullptr;
  base.de = F(T.de_e);
  base.dxs = F(T.dxs);
  base.dxd = F(T.dxd);
  base.dh = F(T.dh);
  base.dmo = F(T.dmo);
  base.dmi = F(T.dmi);
  base.part = F(T.part);
  const int64_t g0 = P.gnn_begin, ng = P.total - P.gnn_begin;
  base.part_stride = ng;
  base.Wc = prm + P.cls1;
  base.Wl = prm + P.cls2;
  base.oc = P.cls1 - g0;
  base.ol = P.cls2 - g0;
  auto stage = [&](bool edges, int j, int64_t p1, int64_t p2) {
    NetStep A = base;
    A.W1 = prm + p1;
    A.W2 = prm + p2;
    A.o1 = p1 - g0;
    A.o2 = p2 - g0;
    A.yh1 = edges ? F(T.yh_e) + j * eH : F(T.yh_n) + j * nH;
    A.yh2 = edges ? F(T.yh_e) + (j + 1) * eH : F(T.yh_n) + (j + 1) * nH;
    A.rs1 = edges ? F(T.rs_e) + j * E : F(T.rs_n) + j * n;
    A.rs2 = edges ? F(T.rs_e) + (j + 1) * E : F(T.rs_n) + (j + 1) * n;
    return A;
  };
  auto node_stage = [&](int k) {
    NetStep A = stage(false, 2 + 2 * k, P.nn1[k], P.nn2[k]);
    A.mo = F(T.mo) + k * nH;
    A.mi = F(T.mi) + k * nH;
    A.h_in = hst(k);
    A.h_out = hst(k + 1);
    A.e_in = est(k);
    return A;
  };
  auto edge_stage = [&](int k) {
    NetStep A = stage(true, 2 + 2 * k, P.en1[k], P.en2[k]);
    A.e_in = est(k);
    A.e_out = est(k + 1);
    A.h_in = hst(k + 1);
    return A;
  };
  NetStep node_enc = stage(false, 0, P.ne1, P.ne2), edge_enc = stage(true, 0, P.ee1, P.ee2);
  node_enc.h_out = hst(0);
  edge_enc.h_in = hst(0);
  edge_enc.e_out = est(0);
  // ---- forward; the last edge update also runs the classifier, forward and backward
  HIPCHK(launch_net(NET_NODE_ENC, node_enc, H, s));
  HIPCHK(launch_net(NET_EDGE_ENC, edge_enc, H, s));
  for (int k = 0; k < S; ++k) {
    HIPCHK(launch_net(NET_NODE, node_stage(k), H, s));
    HIPCHK(launch_net(k + 1 < S ? NET_EDGE : NET_EDGE_LAST, edge_stage(k), H, s));
  }
  // ---- triplets of the purified graph of this step's scores, and the two classifiers on them
  etx_tracks TS{};
  int64_t nrow[2] = {0, 0};
  const int64_t hsz = 3 * (int64_t)H * H + 3 * H + 1;
  float* tprm = ctx->dev_tri_train;
  auto I32 = [&](size_t off) { return reinterpret_cast<int32_t*>(ws + off); };
  if (trip) {
    TS.triplet_capacity = tcap;
    TS.tri_a = I32(X.ta);
    TS.tri_b = I32(X.tb);
    TS.tri_score = F(X.tscore);
    TS.tri_kind = reinterpret_cast<uint8_t*>(ws + X.kind);
    TS.art_off = reinterpret_cast<int64_t*>(ws + X.art_off);
    TS.elb_off = reinterpret_cast<int64_t*>(ws + X.elb_off);
    TS.status = reinterpret_cast<int64_t*>(ws + X.tstatus);
    HIPCHK(launch_triplet_stage(a, TS, ws + X.tri, X.TL, 0));
    int64_t cnt[2];
    HIPCHK(hipMemcpyAsync(&cnt[0], ws + X.tri + X.TL.art_pos + sizeof(int64_t) * n, sizeof(int64_t),
                          hipMemcpyDeviceToHost, s));
    HIPCHK(hipMemcpyAsync(&cnt[1], ws + X.tri + X.TL.elb_pos + sizeof(int64_t) * n, sizeof(int64_t),
                          hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    if (needed) *needed = cnt[0] + cnt[1];
    if (cnt[0] + cnt[1] > tcap) return ETX_ERR_CAPACITY;
    nrow[0] = cnt[0];
    nrow[1] = cnt[1];
    uint8_t* tlab = reinterpret_cast<uint8_t*>(ws + X.lab);
    HIPCHK(launch_tri_labels(a, ws + X.tri, X.TL, TS, *truth, tlab));
    TriTrain R{};
    R.rows[0] = nrow[0];
    R.rows[1] = nrow[1];
    R.prm = tprm;
    R.e = est(S);
    R.tri_a = TS.tri_a;
    R.tri_b = TS.tri_b;
    R.lab = tlab;
    R.alpha = alpha;
    R.gamma = gamma;
    R.dxa = F(X.dxa);
    R.dxb = F(X.dxb);
    R.lpart = F(T.lpart) + kTrainChunks;
    R.part = F(X.part);
    R.part_stride = 2 * hsz;
    HIPCHK(launch_tri_train(R, H, s));
    HIPCHK(launch_tri_edge_grad(a, ws + X.tri, X.TL, TS, F(X.dxa), F(X.dxb), F(T.de_e)));
  }
  // ---- backward
  for (int k = S - 1; k >= 0; --k) {
    NetStep Ae = edge_stage(k), An = node_stage(k);
    if (k == S - 1) Ae.dmo = nullptr;
    An.add_dh = k < S - 1;
    HIPCHK(launch_net(NET_EDGE_BWD, Ae, H, s));
    HIPCHK(launch_net(NET_NODE_BWD, An, H, s));
  }
  node_enc.add_dh = 1;
  HIPCHK(launch_net(NET_EDGE_ENC_BWD, edge_enc, H, s));
  HIPCHK(launch_net(NET_NODE_ENC_BWD, node_enc, H, s));
  // ---- gradients and Adam
  const int64_t nb = (int64_t)blob_floats_of(c);
  const int gn = net_groups(n), ge = net_groups(E);
  GradAdam G{};
  G.set[0].part = F(T.part);
  G.set[0].stride = ng;
  G.set[0].n = ng;
  G.set[0].b0 = P.ee1 - g0;
  G.set[0].b1 = P.nn1[0] - g0;
  G.set[0].b2 = P.cls1 - g0;
  G.set[0].half = P.en1[0] - P.nn1[0];
  G.set[0].g0 = gn;
  G.set[0].g1 = ge;
  G.set[0].grad = grad + g0;
  G.set[0].p = prm + g0;
  G.set[0].m = prm + nb + g0;
  G.set[0].v = prm + 2 * nb + g0;
  G.lr = lr;
  G.loss_part[0] = F(T.lpart);
  G.loss_n[0] = ge;
  if (trip) {
    G.set[1].part = F(X.part);
    G.set[1].stride = G.set[1].n = G.set[1].b1 = 2 * hsz;
    G.set[1].b0 = hsz;
    G.set[1].g0 = net_groups(nrow[0]);
    G.set[1].g1 = net_groups(nrow[1]);
    G.set[1].grad = F(X.tgrad);
    G.set[1].p = tprm;
    G.set[1].m = tprm + 2 * hsz;
    G.set[1].v = tprm + 4 * hsz;
    for (int hd = 0; hd < 2; ++hd) {
      G.loss_part[1 + hd] = F(T.lpart) + (1 + hd) * kTrainChunks;
      G.loss_n[1 + hd] = net_groups(nrow[hd]);
    }
  }
  G.loss = F(T.loss);
  G.loss_dev = loss_dev;
  HIPCHK(launch_grad_adam(G, step, s));
  return ETX_OK;
}

}  // namespace

extern "C" {

etx_status etx_train_gnn_step(etx_ctx* ctx, const etx_hits* hits, etx_out* out, const etx_truth* truth, float alpha,
                              float gamma, float lr, int64_t step, float* loss_dev, void* ws, size_t ws_bytes,
                              etx_stream stream) {
  return gnn_step(ctx, hits, out, truth, alpha, gamma, lr, step, -1, nullptr, loss_dev, ws, ws_bytes, stream);
}

etx_status etx_train_triplet_step(etx_ctx* ctx, const etx_hits* hits, etx_out* out, const etx_truth* truth,
                                  float alpha, float gamma, float lr, int64_t step, int64_t triplet_capacity,
                                  int64_t* triplets_needed, float* loss_dev, void* ws, size_t ws_bytes,
                                  etx_stream stream) {
  if (triplet_capacity < 0) return ETX_ERR_INVALID_ARG;
  return gnn_step(ctx, hits, out, truth, alpha, gamma, lr, step, triplet_capacity, triplets_needed, loss_dev, ws,
                  ws_bytes, stream);
}

}  // extern "C"
