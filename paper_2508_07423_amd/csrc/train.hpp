// Training kernels (train.hip: embedding; train_net.hip: interaction network,
// triplet classifiers, parameter update) and their argument blocks.
#pragma once
#include <cmath>
#include <algorithm>

#include "internal.hpp"

namespace etx {

// Row chunks of a weight gradient: one workgroup and one partial each, added
// in chunk order (a part of the result: another number of chunks gives other
// roundings).
constexpr int kTrainChunks = 256;
// Chunks of `rows` rows that hold any (0 for no rows).
int net_groups(int64_t rows);

// One stage of the network's forward or backward.  Parameters point into the
// FP32 training state in blob order (W[K][H] then b[H]).
struct NetStep {
  int64_t n, E;
  const float *x, *y, *z;          // hits (node encoder)
  float inv_r, inv_z;
  const int64_t *row_ptr, *col_ptr;
  const int32_t *csc, *src, *dst;
  const float *W1, *W2;            // the two layers
  const float *Wc, *Wl;            // classifier: Block and final linear layer (last edge update)
  float *yh1, *rs1, *yh2, *rs2;    // normalised values and reciprocal deviations of both layers
  const float *h_in, *e_in;        // node and edge encodings before the update
  float *h_out, *e_out;            // and after it
  float *mo, *mi;                  // message sums
  uint8_t* lab;                    // edge labels
  const int32_t *succ, *succ2;
  float alpha, gamma;              // focal loss
  float* lpart;                    // [groups] loss partials
  float* score;                    // edge scores (may be null)
  // backward
  float *de, *dxs, *dxd, *dh, *dmo, *dmi;   // dmo null: no message gradients to add
  int add_dh;                      // 0: dh starts from zero
  float* part;                     // [groups][part_stride] gradient partials
  int64_t part_stride;
  int64_t o1, o2, oc, ol;          // parameter offsets of W1, W2, Wc, Wl in a partial
};

enum NetPart {
  NET_NODE_ENC, NET_EDGE_ENC, NET_NODE, NET_EDGE, NET_EDGE_LAST,
  NET_EDGE_BWD, NET_NODE_BWD, NET_EDGE_ENC_BWD, NET_NODE_ENC_BWD
};
hipError_t launch_net(NetPart part, const NetStep& A, int H, hipStream_t s);

// Both triplet classifiers, forward and backward.
struct TriTrain {
  int64_t rows[2];                 // articulations, elbows
  const float* prm;                // both heads: W1[2H][H] b1 W2[H][H] b2 w3[H] b3
  const float* e;                  // e_S
  const int32_t *tri_a, *tri_b;
  const uint8_t* lab;
  float alpha, gamma;
  float *dxa, *dxb;                // [rows][H] gradients of the two input rows
  float* lpart;                    // [2][kTrainChunks]
  float* part;
  int64_t part_stride;
};
hipError_t launch_tri_train(const TriTrain& A, int H, hipStream_t s);

// A parameter range whose partials are added and which takes an Adam step.
// Parameter o has g0 partials below b0, g1 below b1, alternating blocks of
// `half` parameters with g0 and g1 below b2, and g1 after it.
struct GradSet {
  const float* part = nullptr;
  int64_t stride = 0, n = 0;
  int64_t b0 = 0, b1 = 0, b2 = 0, half = 1;
  int g0 = 0, g1 = 0;
  float *grad = nullptr, *p = nullptr, *m = nullptr, *v = nullptr;
};
struct GradAdam {
  GradSet set[2];
  float lr = 0.f, c1 = 1.f, c2 = 1.f;
  const float* loss_part[3] = {};
  int loss_n[3] = {-1, -1, -1};    // partials of loss k; -1: loss k is not written
  float* loss = nullptr;           // [3]
  float* loss_dev = nullptr;       // may be null
  const int64_t* status = nullptr; // may be null; an error there leaves everything as it is
};
hipError_t launch_grad_adam(GradAdam A, int64_t step, hipStream_t s);

// Embedding MLP of the training parameters: forward (every layer's z kept, the
// output to the padded embedding buffer) and backward.
struct EmbTrain {
  int64_t n;
  const float *x, *y, *z;
  float inv_r, inv_z;
  const float* W[5];               // layers 0 .. L (W[K][M] then b[M])
  int64_t o[5];                    // parameter offsets in a partial
  float* zs[4];                    // [n][W]: z of hidden layer l
  float* emb;                      // [n][kDpad]
  const float* de;                 // [n][kDpad] dL/d(embedding)
  int D;
  float* part;
  int64_t part_stride;
  const int64_t* status;
};
hipError_t launch_emb_fwd(const EmbTrain& A, int W, int L, const etx_ctx* c, hipStream_t s);
hipError_t launch_emb_bwd(const EmbTrain& A, int W, int L, hipStream_t s);

constexpr int kHingeBlocks = 512;  // most workgroups of the loss kernels (partials added in block order)
int hinge_blocks(int64_t n);

struct HingeArgs {
  int64_t n;                 // hits
  const float* emb;          // [n][lde]
  int lde;
  const uint8_t* query;      // 1: the hit belongs to a particle with at least three hits
  const int32_t* succ;       // successor hit on the hit's particle (-1: none)
  const int32_t* pred;       // predecessor hit (-1: none)
  const int32_t* particle;   // -1: noise
  const int32_t* rnd;        // random partner of each query (-1: none)
  const int64_t* rnd_ptr;    // [n + 1] random pairs grouped by target: rnd_src[rnd_ptr[b] .. rnd_ptr[b+1]]
  const int32_t* rnd_src;
  const int64_t* row_ptr;    // training radius graph (CSR by source)
  const int32_t* dst;
  const int64_t* col_ptr;    // its CSC
  const int32_t* csc;
  float margin, w_gen;
  float* count_part;         // [kHingeBlocks][2]: genuine and fake pairs per block (counting pass)
  float* loss_part;          // [kHingeBlocks]
  float* g_gen;              // [n][D]
  float* g_rnd;              // [n][D]
  float* g_edge;             // [E][D]
  float* de;                 // [n][ldde]: dL/de per hit
  int ldde;
  const int64_t* status;
};
hipError_t launch_hinge(const HingeArgs& A, int D, hipStream_t s);

int train_net_attributes(size_t max_lds);

}  // namespace etx
