// Training kernels of the interaction network and the triplet classifiers
// (thesis ch. 8 "Graph Neural Network and Classifiers", eq. gnn-loss).
//
// A training step is one event or a few (thousands of rows), so its time is
// the number of kernels in a row and the latency of each.  A kernel therefore
// covers everything that is local to a row (a hit, an edge, a triplet): both
// Blocks of a network forward, or both Blocks backward with their weight
// gradients.  A step is 2 + 2 S launches forward and 2 + 2 S backward (S
// message-passing steps) and one that adds the gradient partials and updates
// the parameters; the classifier's backward is in the last forward launch,
// since it needs nothing from other rows but their number.
//
// Rows are handled in the column layout of tile.hpp (a wave 16 rows, a
// workgroup of four waves 64), products on the FP32 matrix cores with the
// layer's weights in LDS.
//
// Order of additions.  Training is a long chain of steps, and a trained
// network's gradients are small sums of cancelling terms (two FP32 evaluations
// in different orders differ by 1e-5 to 1e-4), so the order is fixed: every
// sum is one chain of fused multiply-adds in index order.
// v_mfma_f32_16x16x4f32 is such a chain over its four K-terms (lane groups 0
// to 3 in turn, rounded after each; checked against fmaf on the GPU over 51,200
// sums of 64 terms), so a product over K runs in index order when lane group g
// supplies term 4 t + g of K-step t: the "natural" layout, four row swaps per
// four registers away from the column layout.  The LayerNorm's sums are such
// products too: with a matrix of ones for a sum over a column, and the
// diagonal of X^T Y for a sum of products.
//
// A weight gradient dW = X^T dZ is a product over rows.  The rows are cut into
// kTrainChunks chunks, one workgroup each (an event's 1,800 hits and 4,600
// edges then fill the chip); the workgroup's dZ goes through LDS (64 rows at a
// time), every wave takes a quarter of the 16-feature blocks of X (read from
// memory as the forward stored it, or recomputed from the stored normalised
// values) and keeps its blocks of dW in accumulators.  Each chunk writes one
// partial per parameter; the parameter update adds them in chunk order.
//
// Measured on one trained event (1,820 hits, 4,600 edges, hidden 32, 4 steps),
// a whole step with its graph: 3,115 -> 306 us (with the triplet classifiers
// 3,910 -> 420 us) against one row per thread with a kernel per layer and a serial
// reduction per layer (of which the reductions took 1,301 us and the forward layers
// 911 us).  The gradients of 61 batches (both hidden sizes, 188 to 50,722 hits) had
// the same bits as those kernels'; the tests compare them with the FP64 oracle.
#include "internal.hpp"
#include "tile.hpp"
#include "train.hpp"

namespace etx {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kRows = kWaves * kCols;       // rows per workgroup tile

// Padded rows in LDS.  kLd: read along a row by both products without (transposed)
// or with little (plain) bank conflict; kLdF: read by the plain product only.
template <int M>
constexpr int kLd = M + 4;
template <int M>
constexpr int kLdF = M + 16;

__device__ inline int lane16() { return threadIdx.x & 15; }

// W[K][M] (row-major, any 4-byte alignment) into LDS rows of LD floats
template <int K, int M, int LD>
__device__ inline void stage_rows(float* l, const float* __restrict__ W) {
#pragma unroll 8
  for (int i = threadIdx.x; i < K * M; i += kThreads) l[(i / M) * LD + i % M] = W[i];
}

// a vector of any 4-byte alignment in column layout / in natural layout
template <int M>
__device__ inline void vec_cols(float* a, const float* __restrict__ b) {
  const int g = lane_group();
#pragma unroll
  for (int r = 0; r < M / 4; ++r) a[r] = b[phi(r, g)];
}
template <int M>
__device__ inline void vec_nat(float* a, const float* __restrict__ b) {
  const int g = lane_group();
#pragma unroll
  for (int r = 0; r < M / 4; ++r) a[r] = b[4 * r + g];
}

// acc[M/4] (column layout) += W^T x for x[K/4] (natural layout)
template <int K, int M, int LD>
__device__ inline void mul_w(float* acc, const float* x, const float* l) {
  const float* w = l + lane_group() * LD + lane16();
  floatx4 c[M / 16];
#pragma unroll
  for (int mb = 0; mb < M / 16; ++mb)
#pragma unroll
    for (int v = 0; v < 4; ++v) c[mb][v] = acc[4 * mb + v];
#pragma unroll
  for (int t = 0; t < K / 4; ++t)
#pragma unroll
    for (int mb = 0; mb < M / 16; ++mb)
      c[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[4 * t * LD + 16 * mb], x[t], c[mb], 0, 0, 0);
#pragma unroll
  for (int mb = 0; mb < M / 16; ++mb)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[4 * mb + v] = c[mb][v];
}

// out[K/4] (column layout) = W dz for dz[M/4] (natural layout)
template <int K, int M>
__device__ inline void mul_wt(float* out, const float* dz, const float* l) {
  const float* w = l + lane16() * kLd<M> + lane_group();
  floatx4 c[K / 16];
#pragma unroll
  for (int kb = 0; kb < K / 16; ++kb) c[kb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < M / 4; ++t)
#pragma unroll
    for (int kb = 0; kb < K / 16; ++kb)
      c[kb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[16 * kb * kLd<M> + 4 * t], dz[t], c[kb], 0, 0, 0);
#pragma unroll
  for (int kb = 0; kb < K / 16; ++kb)
#pragma unroll
    for (int v = 0; v < 4; ++v) out[4 * kb + v] = c[kb][v];
}

// sum over the features of each column (x in natural layout), in every lane
template <int H>
__device__ inline float nat_sum(const float* x) {
  floatx4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < H / 4; ++t) c = __builtin_amdgcn_mfma_f32_16x16x4f32(1.0f, x[t], c, 0, 0, 0);
  return c[0];
}
// sum of x y over the features of each column (both natural), in every lane:
// element (j, j) of X^T Y, which lane group j / 4 holds in register j % 4
template <int H>
__device__ inline float nat_dot(const float* x, const float* y) {
  floatx4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < H / 4; ++t) c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t], y[t], c, 0, 0, 0);
  const int j = lane16();
  const float lo = (j & 1) ? c[1] : c[0], hi = (j & 1) ? c[3] : c[2];
  return __shfl((j & 2) ? hi : lo, 16 * (j >> 2) + j);
}

// z (column layout) -> its normalised value (no ReLU); y (natural layout) its
// ReLU; returns the reciprocal standard deviation
template <int H>
__device__ inline float ln_fwd(float* z, float* y) {
  to_nat<H>(y, z);
  const float mean = nat_sum<H>(y) * (1.0f / H);
#pragma unroll
  for (int r = 0; r < H / 4; ++r) {
    z[r] -= mean;
    y[r] -= mean;
  }
  const float rs = 1.0f / sqrtf(nat_dot<H>(y, y) * (1.0f / H) + 1e-5f);
#pragma unroll
  for (int r = 0; r < H / 4; ++r) {
    z[r] *= rs;
    y[r] = fmaxf(y[r] * rs, 0.f);
  }
  return rs;
}

// dy -> dL/dz through the ReLU and the LayerNorm (d, yh in column layout); dn
// receives it in natural layout
template <int H>
__device__ inline void ln_bwd(float* d, float* dn, const float* yh, float rs) {
  float yn[H / 4];
#pragma unroll
  for (int r = 0; r < H / 4; ++r) d[r] = yh[r] > 0.f ? d[r] : 0.f;
  to_nat<H>(dn, d);
  to_nat<H>(yn, yh);
  const float m = nat_sum<H>(dn) * (1.0f / H), my = nat_dot<H>(dn, yn) * (1.0f / H);
#pragma unroll
  for (int r = 0; r < H / 4; ++r) {
    d[r] = rs * (d[r] - m - yh[r] * my);
    dn[r] = rs * (dn[r] - m - yn[r] * my);
  }
}

// store / load one row in column layout (rows of H floats, 16-byte aligned)
template <int H>
__device__ inline void put(float* base, int64_t row, const float* v, bool valid) {
  store_cols<H>(base + row * H, v, valid);
}
template <int H>
__device__ inline void get(float* v, const float* base, int64_t row) {
  load_cols<H>(v, base + row * H, true);
}

// this wave's 16 rows (column layout) of a workgroup buffer [kRows][kLdF<H>]
template <int H>
__device__ inline void to_lds(float* buf, const float* v) {
  float* row = buf + (wave_id() * kCols + lane16()) * kLdF<H> + 4 * lane_group();
#pragma unroll
  for (int c = 0; c < H / 16; ++c)
    *reinterpret_cast<float4*>(row + 16 * c) = make_float4(v[4 * c], v[4 * c + 1], v[4 * c + 2], v[4 * c + 3]);
}

// acc[mb] += X_block^T dZ over the first nr rows of the workgroup's tile, in
// order: x(r) gives the lane's feature (16 per block) of local row r, dz is the
// workgroup buffer (rows nr .. up to the next multiple of 16 hold zeros)
template <int M, class X>
__device__ inline void wgrad_block(floatx4 (&acc)[M / 16], X x, const float* dz, int nr) {
  const int g = lane_group();
  const float* z = dz + lane16();
  auto step = [&](int r, float xv) {
#pragma unroll
    for (int mb = 0; mb < M / 16; ++mb)
      acc[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv, z[r * kLdF<M> + 16 * mb], acc[mb], 0, 0, 0);
  };
  for (int r0 = 0; r0 < nr; r0 += 16) {
    float xv[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) xv[t] = x(r0 + 4 * t + g);
#pragma unroll
    for (int t = 0; t < 4; ++t) step(r0 + 4 * t + g, xv[t]);
  }
}

// block kb of dW[.][M] into a partial
template <int M>
__device__ inline void put_wgrad(float* dW, int kb, const floatx4 (&acc)[M / 16]) {
  const int g = lane_group();
#pragma unroll
  for (int mb = 0; mb < M / 16; ++mb)
#pragma unroll
    for (int v = 0; v < 4; ++v) dW[(16 * kb + 4 * g + v) * M + 16 * mb + lane16()] = acc[mb][v];
}

// s + feature m of a buffer's first nr rows, in order
template <int M>
__device__ inline float row_sum(float s, const float* buf, int m, int nr) {
#pragma unroll 8
  for (int r = 0; r < nr; ++r) s += buf[r * kLdF<M> + m];
  return s;
}

// The rows of a workgroup: chunk blockIdx.x of `rows` rows.
struct Chunk {
  int64_t begin, end;
  __device__ explicit Chunk(int64_t rows) {
    const int64_t per = (rows + kTrainChunks - 1) / kTrainChunks;
    begin = (int64_t)blockIdx.x * per;
    end = begin + per < rows ? begin + per : rows;
  }
};

// Sigmoid focal loss (Lin et al.) of one logit; d receives dl/dz.
__device__ inline float focal(float z, bool genuine, float alpha, float gamma, float& p, float& d) {
  p = 1.0f / (1.0f + expf(-z));
  const float lp = -(z < 0.f ? -z + log1pf(expf(z)) : log1pf(expf(-z)));     // log p
  const float l1p = -(z > 0.f ? z + log1pf(expf(-z)) : log1pf(expf(z)));     // log (1 - p)
  if (genuine) {
    const float wt = powf(1.f - p, gamma);
    d = alpha * wt * (gamma * p * lp - (1.f - p));
    return -alpha * wt * lp;
  }
  const float wt = powf(p, gamma);
  d = (1.f - alpha) * wt * (p - gamma * (1.f - p) * l1p);
  return -(1.f - alpha) * wt * l1p;
}

// workgroup sum of one value per thread (fixed order), to thread 0
__device__ inline float block_sum(float v, float* tmp) {
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) v += __shfl_xor(v, s);
  if (lane_id() == 0) tmp[wave_id()] = v;
  __syncthreads();
  return (tmp[0] + tmp[1]) + (tmp[2] + tmp[3]);
}

// out += the sum over l's out-edges of a (rows rb .. re-1) plus the sum over its
// in-edges of b, in CSR and CSC order
template <int H>
__device__ inline void add_out(float* out, const float* __restrict__ a, int64_t rb, int64_t re) {
  const int g = lane_group();
#pragma unroll 2
  for (int64_t t = rb; t < re; ++t)
#pragma unroll
    for (int c = 0; c < H / 16; ++c) {
      const float4 v = *reinterpret_cast<const float4*>(a + t * H + 16 * c + 4 * g);
      out[4 * c] += v.x; out[4 * c + 1] += v.y; out[4 * c + 2] += v.z; out[4 * c + 3] += v.w;
    }
}
template <int H>
__device__ inline void add_in(float* out, const float* __restrict__ b, const int32_t* __restrict__ csc, int64_t cb,
                              int64_t ce) {
  const int g = lane_group();
#pragma unroll 2
  for (int64_t t = cb; t < ce; ++t) {
    const float* row = b + (int64_t)csc[t] * H + 4 * g;
#pragma unroll
    for (int c = 0; c < H / 16; ++c) {
      const float4 v = *reinterpret_cast<const float4*>(row + 16 * c);
      out[4 * c] += v.x; out[4 * c + 1] += v.y; out[4 * c + 2] += v.z; out[4 * c + 3] += v.w;
    }
  }
}

// --------------------------------------------------------------------------
// forward
// --------------------------------------------------------------------------

// Two Blocks on a row's input x[K/4] (natural layout): out (column layout) =
// relu(yh2), with yh and rstd of both kept.
template <int K, int H>
__device__ inline void two_blocks(const NetStep& A, const float* w1, const float* w2, const float* x, int64_t row,
                                  bool valid, float* out) {
  float z[H / 4], y[H / 4];
  vec_cols<H>(z, A.W1 + K * H);
  mul_w<K, H, kLdF<H>>(z, x, w1);
  float rs = ln_fwd<H>(z, y);
  put<H>(A.yh1, row, z, valid);
  if (valid && lane_group() == 0) A.rs1[row] = rs;
  vec_cols<H>(z, A.W2 + H * H);
  mul_w<H, H, kLdF<H>>(z, y, w2);
  rs = ln_fwd<H>(z, y);
  put<H>(A.yh2, row, z, valid);
  if (valid && lane_group() == 0) A.rs2[row] = rs;
#pragma unroll
  for (int r = 0; r < H / 4; ++r) out[r] = fmaxf(z[r], 0.f);
}

// node encoder: h0 = Blocks(x/R, y/R, z/Z)
template <int H>
__global__ __launch_bounds__(kThreads) void k_net_node_enc(NetStep A) {
  __shared__ __align__(16) float w2[H * kLdF<H>];
  stage_rows<H, H, kLdF<H>>(w2, A.W2);
  __syncthreads();
  const int g = lane_group();
  for (int64_t t0 = (int64_t)blockIdx.x * kRows; t0 < A.n; t0 += (int64_t)gridDim.x * kRows) {
    const int64_t row = t0 + wave_id() * kCols + lane16();
    const bool valid = row < A.n;
    const int64_t r = valid ? row : A.n - 1;
    const float v0 = A.x[r] * A.inv_r, v1 = A.y[r] * A.inv_r, v2 = A.z[r] * A.inv_z;
    float z[H / 4], y[H / 4];
#pragma unroll
    for (int q = 0; q < H / 4; ++q) {
      const int f = phi(q, g);
      z[q] = fmaf(v2, A.W1[2 * H + f], fmaf(v1, A.W1[H + f], fmaf(v0, A.W1[f], A.W1[3 * H + f])));
    }
    float rs = ln_fwd<H>(z, y);
    put<H>(A.yh1, row, z, valid);
    if (valid && g == 0) A.rs1[row] = rs;
    vec_cols<H>(z, A.W2 + H * H);
    mul_w<H, H, kLdF<H>>(z, y, w2);
    rs = ln_fwd<H>(z, y);
    put<H>(A.yh2, row, z, valid);
    if (valid && g == 0) A.rs2[row] = rs;
#pragma unroll
    for (int q = 0; q < H / 4; ++q) z[q] = fmaxf(z[q], 0.f);
    put<H>(A.h_out, row, z, valid);
  }
}

// edge encoder: e0 = Blocks(h_src, h_dst); also the edge labels (an edge is
// genuine when its target is the source's successor on one of its particles)
template <int H>
__global__ __launch_bounds__(kThreads) void k_net_edge_enc(NetStep A) {
  extern __shared__ __align__(16) float lds[];
  float* w1 = lds;
  float* w2 = w1 + 2 * H * kLdF<H>;
  stage_rows<2 * H, H, kLdF<H>>(w1, A.W1);
  stage_rows<H, H, kLdF<H>>(w2, A.W2);
  __syncthreads();
  for (int64_t t0 = (int64_t)blockIdx.x * kRows; t0 < A.E; t0 += (int64_t)gridDim.x * kRows) {
    const int64_t row = t0 + wave_id() * kCols + lane16();
    const bool valid = row < A.E;
    const int64_t r = valid ? row : A.E - 1;
    const int s = A.src[r], d = A.dst[r];
    if (valid && lane_group() == 0)
      A.lab[row] = (A.succ[s] == d || (A.succ2 && A.succ2[s] == d)) ? 1 : 0;
    float x[2 * H / 4], y[H / 4];
    get<H>(x, A.h_in, s);
    get<H>(x + H / 4, A.h_in, d);
    to_nat<2 * H>(x, x);
    two_blocks<2 * H, H>(A, w1, w2, x, row, valid, y);
    put<H>(A.e_out, row, y, valid);
  }
}

// node update: h <- h + Blocks(h, out-sum, in-sum)
template <int H>
__global__ __launch_bounds__(kThreads) void k_net_node(NetStep A) {
  extern __shared__ __align__(16) float lds[];
  float* w1 = lds;
  float* w2 = w1 + 3 * H * kLdF<H>;
  stage_rows<3 * H, H, kLdF<H>>(w1, A.W1);
  stage_rows<H, H, kLdF<H>>(w2, A.W2);
  __syncthreads();
  for (int64_t t0 = (int64_t)blockIdx.x * kRows; t0 < A.n; t0 += (int64_t)gridDim.x * kRows) {
    const int64_t row = t0 + wave_id() * kCols + lane16();
    const bool valid = row < A.n;
    const int64_t r = valid ? row : A.n - 1;
    const int64_t rb = A.row_ptr[r], re = A.row_ptr[r + 1], cb = A.col_ptr[r], ce = A.col_ptr[r + 1];
    float x[3 * H / 4], xn[3 * H / 4], y[H / 4];
    get<H>(x, A.h_in, r);
#pragma unroll
    for (int q = H / 4; q < 3 * H / 4; ++q) x[q] = 0.f;
    add_out<H>(x + H / 4, A.e_in, rb, re);
    add_in<H>(x + H / 2, A.e_in, A.csc, cb, ce);
    put<H>(A.mo, row, x + H / 4, valid);
    put<H>(A.mi, row, x + H / 2, valid);
    to_nat<3 * H>(xn, x);
    two_blocks<3 * H, H>(A, w1, w2, xn, row, valid, y);
#pragma unroll
    for (int q = 0; q < H / 4; ++q) y[q] += x[q];
    put<H>(A.h_out, row, y, valid);
  }
}

// edge update: e <- e + Blocks(e, h_src, h_dst)
template <int H>
__device__ inline void edge_update(const NetStep& A, const float* w1, const float* w2, int64_t row, bool valid,
                                   float* y) {
  const int64_t r = valid ? row : A.E - 1;
  const int s = A.src[r], d = A.dst[r];
  float x[3 * H / 4], e[H / 4];
  get<H>(e, A.e_in, r);
  get<H>(x + H / 4, A.h_in, s);
  get<H>(x + H / 2, A.h_in, d);
  to_nat<H>(x, e);
  to_nat<2 * H>(x + H / 4, x + H / 4);
  two_blocks<3 * H, H>(A, w1, w2, x, row, valid, y);
#pragma unroll
  for (int q = 0; q < H / 4; ++q) y[q] += e[q];
  put<H>(A.e_out, row, y, valid);
}

template <int H>
__global__ __launch_bounds__(kThreads) void k_net_edge(NetStep A) {
  extern __shared__ __align__(16) float lds[];
  float* w1 = lds;
  float* w2 = w1 + 3 * H * kLdF<H>;
  stage_rows<3 * H, H, kLdF<H>>(w1, A.W1);
  stage_rows<H, H, kLdF<H>>(w2, A.W2);
  __syncthreads();
  for (int64_t t0 = (int64_t)blockIdx.x * kRows; t0 < A.E; t0 += (int64_t)gridDim.x * kRows) {
    const int64_t row = t0 + wave_id() * kCols + lane16();
    float y[H / 4];
    edge_update<H>(A, w1, w2, row, row < A.E, y);
  }
}

// A Block's final linear layer and focal loss, row by row: y (after the ReLU;
// natural layout yn, column layout yc) -> logit -> loss, d = dL/dlogit (0 for
// rows past the end); y and d go to the workgroup's buffers for the layer's
// weight gradient, wv (column layout) receives dL/dy = w d.
template <int H>
__device__ inline float head_loss(const float* yn, const float* yc, const float* __restrict__ w, bool genuine,
                                  bool valid, float alpha, float gamma, float inv_rows, float* ybuf, float* dbuf,
                                  float* wv, float& p, float& d) {
  vec_nat<H>(wv, w);
  floatx4 c;
#pragma unroll
  for (int v = 0; v < 4; ++v) c[v] = w[H];
#pragma unroll
  for (int t = 0; t < H / 4; ++t) c = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[t], yn[t], c, 0, 0, 0);
  const float l = focal(c[0], genuine, alpha, gamma, p, d);
  d = valid ? d * inv_rows : 0.f;
  to_lds<H>(ybuf, yc);
  if (lane_group() == 0) dbuf[wave_id() * kCols + lane16()] = d;
  vec_cols<H>(wv, w);
#pragma unroll
  for (int r = 0; r < H / 4; ++r) wv[r] *= d;
  return valid && lane_group() == 0 ? l : 0.f;
}

// s + sum over the first nr rows of y_r[k] d_r (k < H) or d_r (k == H), in order
template <int H>
__device__ inline float head_grad(float s, const float* ybuf, const float* dbuf, int k, int nr) {
  if (k < H) {
#pragma unroll 8
    for (int r = 0; r < nr; ++r) s = fmaf(ybuf[r * kLdF<H> + k], dbuf[r], s);
  } else {
#pragma unroll 8
    for (int r = 0; r < nr; ++r) s += dbuf[r];
  }
  return s;
}

// The last edge update with the edge classifier, its focal loss and its
// backward: de = dL/de_S, and the classifier's weight gradients.
template <int H>
__global__ __launch_bounds__(kThreads) void k_net_edge_last(NetStep A) {
  extern __shared__ __align__(16) float lds[];
  float* w1 = lds;
  float* w2 = w1 + 3 * H * kLdF<H>;
  float* wc = w2 + H * kLdF<H>;
  float* xb = wc + H * kLd<H>;              // e_S
  float* zb = xb + kRows * kLdF<H>;         // dL/dz of the classifier's Block
  float* yb = w1;                           // its output (in the first layer's place once that is done)
  float* db = zb + kRows * kLdF<H>;         // [kRows] dL/dlogit
  float* tmp = db + kRows;                  // [kWaves]
  stage_rows<H, H, kLd<H>>(wc, A.Wc);
  const int wave = wave_id();
  const float inv_e = 1.0f / (float)A.E;
  floatx4 acc[H / 16];
#pragma unroll
  for (int mb = 0; mb < H / 16; ++mb) acc[mb] = floatx4{0.f, 0.f, 0.f, 0.f};
  float bacc = 0.f, hacc = 0.f, loss = 0.f;
  const Chunk C(A.E);
  for (int64_t t0 = C.begin; t0 < C.end; t0 += kRows) {
    stage_rows<3 * H, H, kLdF<H>>(w1, A.W1);
    if (t0 == C.begin) stage_rows<H, H, kLdF<H>>(w2, A.W2);
    __syncthreads();
    const int nr = (int)min((int64_t)kRows, C.end - t0);
    const int64_t row = t0 + wave * kCols + lane16();
    const bool live = wave * kCols < nr, valid = row < C.end;
    float e[H / 4], z[H / 4], y[H / 4], wv[H / 4], dn[H / 4];
    float rs = 0.f;
    if (live) {
      edge_update<H>(A, w1, w2, row, valid, e);
      to_lds<H>(xb, e);
      to_nat<H>(e, e);
      vec_cols<H>(z, A.Wc + H * H);
      mul_w<H, H, kLd<H>>(z, e, wc);
      rs = ln_fwd<H>(z, y);
    }
    __syncthreads();                        // every wave is past the first layer's weights
    if (live) {
#pragma unroll
      for (int r = 0; r < H / 4; ++r) e[r] = fmaxf(z[r], 0.f);
      float p, d;
      loss += head_loss<H>(y, e, A.Wl, valid && A.lab[row] != 0, valid, A.alpha, A.gamma, inv_e, yb, db, wv, p, d);
      if (A.score && valid && lane_group() == 0) A.score[row] = p;
      ln_bwd<H>(wv, dn, z, rs);
      to_lds<H>(zb, wv);
      mul_wt<H, H>(e, dn, wc);
      put<H>(A.de, row, e, valid);
    }
    __syncthreads();
    if (wave < H / 16) wgrad_block<H>(acc, [&](int r) { return xb[r * kLdF<H> + 16 * wave + lane16()]; }, zb, nr);
    const int t = threadIdx.x;
    if (t < H) bacc = row_sum<H>(bacc, zb, t, nr);
    else if (t <= 2 * H) hacc = head_grad<H>(hacc, yb, db, t - H, nr);
    __syncthreads();
  }
  float* part = A.part + (int64_t)blockIdx.x * A.part_stride;
  if (wave < H / 16) put_wgrad<H>(part + A.oc, wave, acc);
  const int t = threadIdx.x;
  if (t < H) part[A.oc + H * H + t] = bacc;
  else if (t <= 2 * H) part[A.ol + t - H] = hacc;
  loss = block_sum(loss, tmp);
  if (t == 0) A.lpart[blockIdx.x] = loss * inv_e;
}

// --------------------------------------------------------------------------
// backward
// --------------------------------------------------------------------------

// Gradients of two Blocks from dy[H/4] (column layout, overwritten): dx[K/4] =
// dL/dx, the rows' dL/dz of both layers in the workgroup buffers.
template <int K, int H>
__device__ inline void two_blocks_bwd(const NetStep& A, const float* w1, const float* w2, int64_t r, bool valid,
                                      float* dy, float* dx, float* z1b, float* z2b) {
  float yh[H / 4], da[H / 4], dn[H / 4];
  get<H>(yh, A.yh2, r);
  if (!valid) {
#pragma unroll
    for (int q = 0; q < H / 4; ++q) dy[q] = 0.f;
  }
  ln_bwd<H>(dy, dn, yh, A.rs2[r]);
  to_lds<H>(z2b, dy);
  mul_wt<H, H>(da, dn, w2);
  get<H>(yh, A.yh1, r);
  ln_bwd<H>(da, dn, yh, A.rs1[r]);
  to_lds<H>(z1b, da);
  if constexpr (K > 0) mul_wt<K, H>(dx, dn, w1);
}

// Weight gradients of two Blocks over one workgroup tile: 16-feature blocks q
// = wave, wave + 4, ... of layer 1's K inputs (x1(q, r)) and then of layer 2's
// H inputs (the ReLU of yh1).  Rows past the end have zero dL/dz.
template <int K, int H>
struct BlocksGrad {
  static constexpr int N1 = K / 16, N = N1 + H / 16, NI = (N + kWaves - 1) / kWaves;
  floatx4 acc[NI][H / 16];
  float bias = 0.f;
  __device__ BlocksGrad() {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int mb = 0; mb < H / 16; ++mb) acc[i][mb] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  template <class X1>
  __device__ void add(X1 x1, const float* yh1, int64_t t0, int64_t rows, int nr, const float* z1b, const float* z2b) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int q = wave_id() + kWaves * i;
      if (q < N1) {
        wgrad_block<H>(acc[i], [&](int r) { return x1(q, r); }, z1b, nr);
      } else if (q < N) {
        const float* y = yh1 + 16 * (q - N1) + lane16();
        wgrad_block<H>(acc[i], [&](int r) { return fmaxf(y[min(t0 + r, rows - 1) * H], 0.f); }, z2b, nr);
      }
    }
    const int t = threadIdx.x;
    if (t < H) bias = row_sum<H>(bias, z1b, t, nr);
    else if (t < 2 * H) bias = row_sum<H>(bias, z2b, t - H, nr);
  }
  // layer 1's parameters at p1 (Kw rows, then the bias), layer 2's at p2
  __device__ void store(float* p1, int Kw, float* p2) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int q = wave_id() + kWaves * i;
      if (q < N1) put_wgrad<H>(p1, q, acc[i]);
      else if (q < N) put_wgrad<H>(p2, q - N1, acc[i]);
    }
    const int t = threadIdx.x;
    if (t < H) p1[Kw * H + t] = bias;
    else if (t < 2 * H) p2[H * H + t - H] = bias;
  }
};

// Edge rows: de <- dL/de of the update's output (de, plus the message
// gradients of the node update after it when dmo is set); the update's
// gradient adds its input part to de and writes dxs, dxd for the node rows.
// ENC: the edge encoder, whose input is [h_src, h_dst].
template <int H, bool ENC>
__global__ __launch_bounds__(kThreads) void k_net_edge_bwd(NetStep A) {
  constexpr int K = ENC ? 2 * H : 3 * H;
  extern __shared__ __align__(16) float lds[];
  float* w1 = lds;
  float* w2 = w1 + K * kLd<H>;
  float* z1b = w2 + H * kLd<H>;
  float* z2b = z1b + kRows * kLdF<H>;
  int* sb = reinterpret_cast<int*>(z2b + kRows * kLdF<H>);  // [kRows] sources
  int* db = sb + kRows;                                     // [kRows] targets
  stage_rows<K, H, kLd<H>>(w1, A.W1);
  stage_rows<H, H, kLd<H>>(w2, A.W2);
  __syncthreads();
  BlocksGrad<K, H> G;
  const Chunk C(A.E);
  for (int64_t t0 = C.begin; t0 < C.end; t0 += kRows) {
    const int nr = (int)min((int64_t)kRows, C.end - t0);
    const int64_t row = t0 + wave_id() * kCols + lane16();
    const bool valid = row < C.end;
    const int64_t r = valid ? row : C.end - 1;
    const int s = A.src[r], d = A.dst[r];
    if (lane_group() == 0) {
      sb[wave_id() * kCols + lane16()] = s;
      db[wave_id() * kCols + lane16()] = d;
    }
    if (wave_id() * kCols < nr) {
    float de[H / 4], dy[H / 4], dx[K / 4];
    get<H>(de, A.de, r);
    if (A.dmo) {
      get<H>(dy, A.dmo, s);
      get<H>(dx, A.dmi, d);
#pragma unroll
      for (int q = 0; q < H / 4; ++q) de[q] += dy[q] + dx[q];
    }
#pragma unroll
    for (int q = 0; q < H / 4; ++q) dy[q] = de[q];
    two_blocks_bwd<K, H>(A, w1, w2, r, valid, dy, dx, z1b, z2b);
    if constexpr (!ENC) {
#pragma unroll
      for (int q = 0; q < H / 4; ++q) de[q] += dx[q];
      put<H>(A.de, row, de, valid);
    }
    put<H>(A.dxs, row, dx + (K - 2 * H) / 4, valid);
    put<H>(A.dxd, row, dx + (K - H) / 4, valid);
    }
    __syncthreads();
    auto x1 = [&](int q, int rr) {
      const int seg = ENC ? q / (H / 16) + 1 : q / (H / 16), f = 16 * (q % (H / 16)) + lane16();
      const float* base = seg == 0 ? A.e_in + min(t0 + rr, C.end - 1) * H
                                   : A.h_in + (int64_t)(seg == 1 ? sb[rr] : db[rr]) * H;
      return base[f];
    };
    G.add(x1, A.yh1, t0, C.end, nr, z1b, z2b);
    __syncthreads();
  }
  float* part = A.part + (int64_t)blockIdx.x * A.part_stride;
  G.store(part + A.o1, K, part + A.o2);
}

// Node rows: dh <- dL/dh of the update's output (dh when add_dh is set, plus
// the edge rows' dxs over out-edges and dxd over in-edges); the update's
// gradient adds its input part to dh and writes dmo, dmi for the edge rows.
template <int H>
__global__ __launch_bounds__(kThreads) void k_net_node_bwd(NetStep A) {
  constexpr int K = 3 * H;
  extern __shared__ __align__(16) float lds[];
  float* w1 = lds;
  float* w2 = w1 + K * kLd<H>;
  float* z1b = w2 + H * kLd<H>;
  float* z2b = z1b + kRows * kLdF<H>;
  stage_rows<K, H, kLd<H>>(w1, A.W1);
  stage_rows<H, H, kLd<H>>(w2, A.W2);
  __syncthreads();
  BlocksGrad<K, H> G;
  const Chunk C(A.n);
  for (int64_t t0 = C.begin; t0 < C.end; t0 += kRows) {
    const int nr = (int)min((int64_t)kRows, C.end - t0);
    const int64_t row = t0 + wave_id() * kCols + lane16();
    const bool valid = row < C.end;
    const int64_t r = valid ? row : C.end - 1;
    const int64_t rb = A.row_ptr[r], re = A.row_ptr[r + 1], cb = A.col_ptr[r], ce = A.col_ptr[r + 1];
    if (wave_id() * kCols < nr) {
    float dh[H / 4], dy[H / 4], dx[K / 4];
#pragma unroll
    for (int q = 0; q < H / 4; ++q) dh[q] = 0.f;
    if (A.add_dh) get<H>(dh, A.dh, r);
    add_out<H>(dh, A.dxs, rb, re);
    add_in<H>(dh, A.dxd, A.csc, cb, ce);
#pragma unroll
    for (int q = 0; q < H / 4; ++q) dy[q] = dh[q];
    two_blocks_bwd<K, H>(A, w1, w2, r, valid, dy, dx, z1b, z2b);
#pragma unroll
    for (int q = 0; q < H / 4; ++q) dh[q] += dx[q];
    put<H>(A.dh, row, dh, valid);
    put<H>(A.dmo, row, dx + H / 4, valid);
    put<H>(A.dmi, row, dx + H / 2, valid);
    }
    __syncthreads();
    auto x1 = [&](int q, int rr) {
      const int seg = q / (H / 16), f = 16 * (q % (H / 16)) + lane16();
      const float* base = seg == 0 ? A.h_in : seg == 1 ? A.mo : A.mi;
      return base[min(t0 + rr, C.end - 1) * H + f];
    };
    G.add(x1, A.yh1, t0, C.end, nr, z1b, z2b);
    __syncthreads();
  }
  float* part = A.part + (int64_t)blockIdx.x * A.part_stride;
  G.store(part + A.o1, K, part + A.o2);
}

// node encoder
template <int H>
__global__ __launch_bounds__(kThreads) void k_net_node_enc_bwd(NetStep A) {
  extern __shared__ __align__(16) float lds[];
  float* w2 = lds;
  float* z1b = w2 + H * kLd<H>;
  float* z2b = z1b + kRows * kLdF<H>;
  float* cb3 = z2b + kRows * kLdF<H>;       // [3][kRows] inputs
  stage_rows<H, H, kLd<H>>(w2, A.W2);
  __syncthreads();
  BlocksGrad<0, H> G;
  float in_acc = 0.f;                       // thread t < 3 H: dW1[t / H][t % H]
  const Chunk C(A.n);
  for (int64_t t0 = C.begin; t0 < C.end; t0 += kRows) {
    const int nr = (int)min((int64_t)kRows, C.end - t0);
    const int local = wave_id() * kCols + lane16();
    const int64_t row = t0 + local;
    const bool valid = row < C.end;
    const int64_t r = valid ? row : C.end - 1;
    const int64_t rb = A.row_ptr[r], re = A.row_ptr[r + 1], cb = A.col_ptr[r], ce = A.col_ptr[r + 1];
    if (lane_group() == 0) {
      cb3[local] = A.x[r] * A.inv_r;
      cb3[kRows + local] = A.y[r] * A.inv_r;
      cb3[2 * kRows + local] = A.z[r] * A.inv_z;
    }
    if (wave_id() * kCols < nr) {
      float dh[H / 4];
#pragma unroll
      for (int q = 0; q < H / 4; ++q) dh[q] = 0.f;
      if (A.add_dh) get<H>(dh, A.dh, r);
      add_out<H>(dh, A.dxs, rb, re);
      add_in<H>(dh, A.dxd, A.csc, cb, ce);
      two_blocks_bwd<0, H>(A, nullptr, w2, r, valid, dh, nullptr, z1b, z2b);
    }
    __syncthreads();
    G.add([](int, int) { return 0.f; }, A.yh1, t0, C.end, nr, z1b, z2b);
    if (const int o = threadIdx.x; o < 3 * H) {
      const float* c = cb3 + (o / H) * kRows;
#pragma unroll 8
      for (int q = 0; q < nr; ++q) in_acc = fmaf(c[q], z1b[q * kLdF<H> + o % H], in_acc);
    }
    __syncthreads();
  }
  static_assert(3 * H <= kThreads, "one input-layer weight per thread");
  float* part = A.part + (int64_t)blockIdx.x * A.part_stride;
  G.store(part + A.o1, 3, part + A.o2);
  if (threadIdx.x < 3 * H) part[A.o1 + threadIdx.x] = in_acc;
}

// --------------------------------------------------------------------------
// triplet classifiers: forward, loss and backward of a row in one kernel
// (everything but the gather of e_S is local to the row).  blockIdx.y picks
// the classifier: 0 articulations (rows 0 .. n[0]-1), 1 elbows (after them).
// --------------------------------------------------------------------------
template <int H>
__global__ __launch_bounds__(kThreads) void k_tri_train(TriTrain A) {
  constexpr int K = 2 * H;
  constexpr int64_t kHead = 3 * H * H + 3 * H + 1;
  const int hd = blockIdx.y;
  const int64_t rows = A.rows[hd], r0 = hd ? A.rows[0] : 0;
  const Chunk C(rows);
  if (C.begin >= rows) return;
  extern __shared__ __align__(16) float lds[];
  float* w1 = lds;
  float* w2 = w1 + K * kLd<H>;
  float* xb = w2 + H * kLd<H>;              // layer 2's input
  float* z1b = xb + kRows * kLdF<H>;
  float* z2b = z1b + kRows * kLdF<H>;
  float* yb = z2b + kRows * kLdF<H>;        // layer 3's input
  float* db = yb + kRows * kLdF<H>;         // [kRows]
  float* tmp = db + kRows;                  // [kWaves]
  int* ab = reinterpret_cast<int*>(tmp + kWaves);   // [kRows] first edges
  int* bb = ab + kRows;                             // [kRows] second edges
  const float* P = A.prm + hd * kHead;      // W1 b1 W2 b2 w3 b3
  const float* W2 = P + K * H + H;
  const float* W3 = W2 + H * H + H;
  stage_rows<K, H, kLd<H>>(w1, P);
  stage_rows<H, H, kLd<H>>(w2, W2);
  __syncthreads();
  const int wave = wave_id();
  const float inv_rows = 1.0f / (float)rows;
  constexpr int N1 = K / 16, N = N1 + H / 16, NI = (N + kWaves - 1) / kWaves;
  floatx4 acc[NI][H / 16];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int mb = 0; mb < H / 16; ++mb) acc[i][mb] = floatx4{0.f, 0.f, 0.f, 0.f};
  float bacc = 0.f, bacc2 = 0.f, loss = 0.f;
  for (int64_t t0 = C.begin; t0 < C.end; t0 += kRows) {
    const int nr = (int)min((int64_t)kRows, C.end - t0);
    const int local = wave * kCols + lane16();
    const int64_t row = t0 + local;
    const bool valid = row < C.end;
    const int64_t r = r0 + (valid ? row : C.end - 1);
    const int ea = A.tri_a[r], eb = A.tri_b[r];
    if (lane_group() == 0) {
      ab[local] = ea;
      bb[local] = eb;
    }
    if (wave * kCols < nr) {
      float x[K / 4], yh1[H / 4], yh2[H / 4], y[H / 4], yn[H / 4], wv[H / 4];
      get<H>(x, A.e, ea);
      get<H>(x + H / 4, A.e, eb);
      to_nat<K>(x, x);
      vec_cols<H>(yh1, P + K * H);
      mul_w<K, H, kLd<H>>(yh1, x, w1);
      const float rs1 = ln_fwd<H>(yh1, yn);
#pragma unroll
      for (int q = 0; q < H / 4; ++q) y[q] = fmaxf(yh1[q], 0.f);
      to_lds<H>(xb, y);
      vec_cols<H>(yh2, W2 + H * H);
      mul_w<H, H, kLd<H>>(yh2, yn, w2);
      const float rs2 = ln_fwd<H>(yh2, yn);
#pragma unroll
      for (int q = 0; q < H / 4; ++q) y[q] = fmaxf(yh2[q], 0.f);
      float p, d;
      loss += head_loss<H>(yn, y, W3, valid && A.lab[r] != 0, valid, A.alpha, A.gamma, inv_rows, yb, db, wv, p, d);
      ln_bwd<H>(wv, yn, yh2, rs2);
      to_lds<H>(z2b, wv);
      mul_wt<H, H>(y, yn, w2);
      ln_bwd<H>(y, yn, yh1, rs1);
      to_lds<H>(z1b, y);
      mul_wt<K, H>(x, yn, w1);
      put<H>(A.dxa, r, x, valid);
      put<H>(A.dxb, r, x + H / 4, valid);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int q = wave + kWaves * i;
      if (q < N1) {
        const int* id = q < H / 16 ? ab : bb;
        const float* base = A.e + 16 * (q % (H / 16)) + lane16();
        wgrad_block<H>(acc[i], [&](int rr) { return base[(int64_t)id[rr] * H]; }, z1b, nr);
      } else if (q < N) {
        const float* base = xb + 16 * (q - N1) + lane16();
        wgrad_block<H>(acc[i], [&](int rr) { return base[rr * kLdF<H>]; }, z2b, nr);
      }
    }
    const int t = threadIdx.x;
    if (t < H) bacc = row_sum<H>(bacc, z1b, t, nr);
    else if (t < 2 * H) bacc = row_sum<H>(bacc, z2b, t - H, nr);
    if (t <= H) bacc2 = head_grad<H>(bacc2, yb, db, t, nr);
    __syncthreads();
  }
  float* part = A.part + (int64_t)blockIdx.x * A.part_stride + hd * kHead;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int q = wave + kWaves * i;
    if (q < N1) put_wgrad<H>(part, q, acc[i]);
    else if (q < N) put_wgrad<H>(part + K * H + H, q - N1, acc[i]);
  }
  const int t = threadIdx.x;
  if (t < H) part[K * H + t] = bacc;
  else if (t < 2 * H) part[K * H + H + H * H + t - H] = bacc;
  if (t <= H) part[K * H + H + H * H + H + t] = bacc2;
  loss = block_sum(loss, tmp);
  if (t == 0) A.lpart[hd * kTrainChunks + blockIdx.x] = loss * inv_rows;
}

// --------------------------------------------------------------------------
// gradient partials -> gradient -> Adam, and the loss sums
// --------------------------------------------------------------------------

// One thread per parameter adds its partials in chunk order and takes the
// Adam step (beta1 0.9, beta2 0.999) when lr > 0.  The additions are a chain,
// the loads are not: kAhead of them are in flight.  The last workgroup adds
// the loss partials.
constexpr int kAhead = 32;
constexpr int kAdamThreads = 64;

__global__ __launch_bounds__(kAdamThreads) void k_grad_adam(GradAdam A) {
  if (A.status && A.status[0] != 0) return;
  const int t = threadIdx.x;
  int64_t b = blockIdx.x;
  if (b == (int64_t)gridDim.x - 1) {
    for (int k = 0; k < 3; ++k) {
      if (A.loss_n[k] < 0) continue;
      float s = 0.f;
      for (int i = t; i < A.loss_n[k]; i += kAdamThreads) s += A.loss_part[k][i];
#pragma unroll
      for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d);
      if (t == 0) {
        A.loss[k] = s;
        if (A.loss_dev) A.loss_dev[k] = s;
      }
    }
    return;
  }
  int j = 0;
  const int64_t b0 = (A.set[0].n + kAdamThreads - 1) / kAdamThreads;
  if (b >= b0) {
    b -= b0;
    j = 1;
  }
  const GradSet& S = A.set[j];
  const int64_t o = b * kAdamThreads + t;
  if (o >= S.n) return;
  const int G = o < S.b0 ? S.g0 : o < S.b1 ? S.g1 : o < S.b2 ? ((o - S.b1) / S.half % 2 ? S.g1 : S.g0) : S.g1;
  const float* p = S.part + o;
  float g = 0.f;
  for (int c = 0; c < G; c += kAhead) {
    float v[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) v[u] = c + u < G ? p[(int64_t)(c + u) * S.stride] : 0.f;
#pragma unroll
    for (int u = 0; u < kAhead; ++u) g += v[u];
  }
  S.grad[o] = g;
  if (!(A.lr > 0.f)) return;
  const float b1 = 0.9f, b2 = 0.999f;
  const float mi = b1 * S.m[o] + (1.f - b1) * g;
  const float vi = b2 * S.v[o] + (1.f - b2) * g * g;
  S.m[o] = mi;
  S.v[o] = vi;
  S.p[o] -= A.lr * (mi / A.c1) / (sqrtf(vi / A.c2) + 1e-8f);
}

// LDS of `wf` weight rows read by the forward product only, `w` others and `bufs` workgroup buffers
template <int H>
constexpr size_t lds_bytes(int wf, int w, int bufs, int words = 0) {
  return sizeof(float) * ((size_t)wf * kLdF<H> + (size_t)w * kLd<H> + (size_t)bufs * kRows * kLdF<H> + words);
}

}  // namespace

// --------------------------------------------------------------------------
// launchers
// --------------------------------------------------------------------------

int net_groups(int64_t rows) {
  const int64_t per = (rows + kTrainChunks - 1) / kTrainChunks;
  return rows > 0 ? (int)((rows + per - 1) / per) : 0;
}

hipError_t launch_net(NetPart part, const NetStep& A, int H, hipStream_t s) {
  const bool edges = part == NET_EDGE_ENC || part == NET_EDGE || part == NET_EDGE_LAST || part == NET_EDGE_BWD ||
                     part == NET_EDGE_ENC_BWD;
  const int64_t rows = edges ? A.E : A.n;
  if (rows == 0) return hipSuccess;
  // forward: 64 rows per workgroup; backward: one chunk per workgroup
  const dim3 fwd((unsigned)std::min<int64_t>((rows + kRows - 1) / kRows, 1024)), bwd((unsigned)net_groups(rows));
#define NET(grid_, k32_, k64_, ...)                                                                     \
  if (H == 32) hipLaunchKernelGGL((k32_), grid_, dim3(kThreads), lds_bytes<32>(__VA_ARGS__), s, A);      \
  else if (H == 64) hipLaunchKernelGGL((k64_), grid_, dim3(kThreads), lds_bytes<64>(__VA_ARGS__), s, A); \
  else return hipErrorInvalidValue;                                                                     \
  return hipGetLastError();
  switch (part) {
    case NET_NODE_ENC: NET(fwd, k_net_node_enc<32>, k_net_node_enc<64>, 0, 0, 0)
    case NET_EDGE_ENC: NET(fwd, k_net_edge_enc<32>, k_net_edge_enc<64>, 3 * H, 0, 0)
    case NET_NODE: NET(fwd, k_net_node<32>, k_net_node<64>, 4 * H, 0, 0)
    case NET_EDGE: NET(fwd, k_net_edge<32>, k_net_edge<64>, 4 * H, 0, 0)
    case NET_EDGE_LAST: NET(bwd, k_net_edge_last<32>, k_net_edge_last<64>, 4 * H, H, 2, kRows + kWaves)
    case NET_EDGE_BWD: NET(bwd, (k_net_edge_bwd<32, false>), (k_net_edge_bwd<64, false>), 0, 4 * H, 2, 2 * kRows)
    case NET_NODE_BWD: NET(bwd, k_net_node_bwd<32>, k_net_node_bwd<64>, 0, 4 * H, 2)
    case NET_EDGE_ENC_BWD: NET(bwd, (k_net_edge_bwd<32, true>), (k_net_edge_bwd<64, true>), 0, 3 * H, 2, 2 * kRows)
    case NET_NODE_ENC_BWD: NET(bwd, k_net_node_enc_bwd<32>, k_net_node_enc_bwd<64>, 0, H, 2, 3 * kRows)
  }
#undef NET
  return hipErrorInvalidValue;
}

hipError_t launch_tri_train(const TriTrain& A, int H, hipStream_t s) {
  const dim3 grid((unsigned)std::max(net_groups(A.rows[0]), net_groups(A.rows[1])), 2);
  if (grid.x == 0) return hipSuccess;
  if (H == 32)
    hipLaunchKernelGGL(k_tri_train<32>, grid, dim3(kThreads), lds_bytes<32>(0, 3 * H, 4, 3 * kRows + kWaves), s, A);
  else if (H == 64)
    hipLaunchKernelGGL(k_tri_train<64>, grid, dim3(kThreads), lds_bytes<64>(0, 3 * H, 4, 3 * kRows + kWaves), s, A);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_grad_adam(GradAdam A, int64_t step, hipStream_t s) {
  A.c1 = (float)(1.0 - std::pow(0.9, (double)step));
  A.c2 = (float)(1.0 - std::pow(0.999, (double)step));
  const int64_t blocks = (A.set[0].n + kAdamThreads - 1) / kAdamThreads + (A.set[1].n + kAdamThreads - 1) / kAdamThreads + 1;
  hipLaunchKernelGGL(k_grad_adam, dim3((unsigned)blocks), dim3(kAdamThreads), 0, s, A);
  return hipGetLastError();
}

int train_net_attributes(size_t max_lds) {
  int bad = 0;
  auto set = [&](const void* f) {
    bad |= hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)max_lds) != hipSuccess;
  };
#define SET(H_)                                                   \
  set(reinterpret_cast<const void*>(k_net_edge_enc<H_>));         \
  set(reinterpret_cast<const void*>(k_net_node<H_>));             \
  set(reinterpret_cast<const void*>(k_net_edge<H_>));             \
  set(reinterpret_cast<const void*>(k_net_edge_last<H_>));        \
  set(reinterpret_cast<const void*>(k_net_edge_bwd<H_, false>));  \
  set(reinterpret_cast<const void*>(k_net_edge_bwd<H_, true>));   \
  set(reinterpret_cast<const void*>(k_net_node_bwd<H_>));         \
  set(reinterpret_cast<const void*>(k_net_node_enc_bwd<H_>));     \
  set(reinterpret_cast<const void*>(k_tri_train<H_>));
  SET(32)
  SET(64)
#undef SET
  return bad;
}

}  // namespace etx
