// In-library training of the embedding MLP (thesis ch. 8 "Hit Embedding and
// Rough Graph Construction", eqs. loss1-loss3): the forward that keeps what
// the backward needs, the pairwise hinge loss, and the backward with its
// weight gradients.
//
// The forward builds the training graph, whose edges are decided by single
// bits of the embedding, so every output is one chain of multiply-adds over
// its inputs in order, starting from the bias.  The backward is products on
// the FP32 matrix cores in the column layout of tile.hpp; weight gradients are
// one partial per workgroup, added in a fixed order by the parameter update
// (train_net.hip), so a step is bitwise reproducible.
#include "internal.hpp"
#include "tile.hpp"
#include "train.hpp"

namespace etx {

namespace {

constexpr int kThreads = 256;

// Sixteen hits per workgroup, sixteen threads per hit: a thread holds W / 16
// outputs of its hit, the hit's inputs are read from LDS (broadcast within the
// row's threads), the layer's weights from LDS in 16-byte chunks.  All layers
// of the 16 hits run in one launch; a one-event batch (about 1,800 hits) fills
// 114 workgroups.
constexpr int kEmbRows = 16;

template <int N>
__device__ inline void fma_row(float* z, float x, const float* w) {
#pragma unroll
  for (int m = 0; m < N; ++m) z[m] = fmaf(x, w[m], z[m]);
}

template <int W>
__global__ __launch_bounds__(kThreads) void k_emb_fwd(EmbTrain A, int L) {
  if (A.status[0] != 0) return;
  constexpr int N = W / 16;                // outputs per thread
  constexpr int LDX = W + 4;
  extern __shared__ __align__(16) float lds[];
  float* w = lds;                          // [W][W]
  float* xs = w + W * W;                   // [2][kEmbRows][LDX]
  const int r = threadIdx.x >> 4, c = threadIdx.x & 15;
  for (int64_t t0 = (int64_t)blockIdx.x * kEmbRows; t0 < A.n; t0 += (int64_t)gridDim.x * kEmbRows) {
    const int64_t row = t0 + r;
    const bool valid = row < A.n;
    const int64_t i = valid ? row : A.n - 1;
    float in[3];
    in[0] = hypotf(A.x[i], A.y[i]) * A.inv_r;
    in[1] = atan2f(A.y[i], A.x[i]) * (1.0f / 3.14159265358979f);
    in[2] = A.z[i] * A.inv_z;
    float z[N];
    // layer 0: output m = c N + q
    {
      const float* W0 = A.W[0];
#pragma unroll
      for (int q = 0; q < N; ++q) z[q] = W0[3 * W + c * N + q];
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int q = 0; q < N; ++q) z[q] = fmaf(in[k], W0[k * W + c * N + q], z[q]);
    }
    for (int l = 0; l < L; ++l) {
      float* xb = xs + (l & 1) * kEmbRows * LDX + r * LDX;
#pragma unroll
      for (int q = 0; q < N; ++q) {
        if (valid) A.zs[l][row * W + c * N + q] = z[q];
        xb[c * N + q] = fmaxf(z[q], 0.f);
      }
      const float* Wn = A.W[l + 1];
      if (l + 1 < L) {
#pragma unroll 8
        for (int k = threadIdx.x; k < W * W; k += kThreads) w[k] = Wn[k];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < N; ++q) z[q] = Wn[W * W + c * N + q];
#pragma unroll 8
        for (int k = 0; k < W; ++k) fma_row<N>(z, xb[k], w + k * W + c * N);
      } else {
        for (int k = threadIdx.x; k < W * A.D; k += kThreads) w[k] = Wn[k];
        __syncthreads();
        float o = 0.f;
        if (c < A.D) {
          o = Wn[W * A.D + c];
#pragma unroll 8
          for (int k = 0; k < W; ++k) o = fmaf(xb[k], w[k * A.D + c], o);
        }
        if (valid) A.emb[row * kDpad + c] = o;
      }
      __syncthreads();                     // the next layer's (or tile's) weights replace these
    }
  }
}

// Backward: one chunk of hits per workgroup (see train_net.hip: chunks, order
// of additions, natural layout), layer by layer from the output; the layer's
// dL/dz goes through one LDS buffer for its weight gradient, its weights
// replace the previous layer's.
constexpr int kRows = 64;

template <int W, int L>
__global__ __launch_bounds__(kThreads) void k_emb_bwd(EmbTrain A) {
  if (A.status[0] != 0) return;
  constexpr int LD = W + 4, LDZ = W + 16, LDO = 16 + 4, NI = (W / 16 + 3) / 4, MB = W / 16;
  constexpr int NIN = (3 * W + kThreads - 1) / kThreads;
  extern __shared__ __align__(16) float lds[];
  float* w = lds;                          // [W][LD] (the output layer: [W][LDO], columns past D zero)
  float* zb = w + W * LD;                  // [kRows][LDZ] (the output layer: [kRows][LDO])
  float* cyl = zb + kRows * LDZ;           // [3][kRows]
  const int lane = lane_id(), g = lane_group(), j = lane & 15, wave = wave_id(), t = threadIdx.x;
  const int local = wave * kCols + j;
  floatx4 acc_o[NI], acc_h[L > 1 ? L - 1 : 1][NI][MB];
  float bias[L + 1], in_acc[NIN];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    acc_o[i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int l = 0; l < L - 1; ++l)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) acc_h[l][i][mb] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int l = 0; l <= L; ++l) bias[l] = 0.f;
#pragma unroll
  for (float& v : in_acc) v = 0.f;
  const int64_t per = (A.n + kTrainChunks - 1) / kTrainChunks;
  const int64_t begin = (int64_t)blockIdx.x * per, end = min(begin + per, A.n);
  for (int64_t t0 = begin; t0 < end; t0 += kRows) {
    const int nr = (int)min((int64_t)kRows, end - t0);
    const bool live = wave * kCols < nr;
    const int64_t row = t0 + local;
    const bool valid = row < end;
    const int64_t r = valid ? row : end - 1;
    if (g == 0) {
      cyl[local] = hypotf(A.x[r], A.y[r]) * A.inv_r;
      cyl[kRows + local] = atan2f(A.y[r], A.x[r]) * (1.0f / 3.14159265358979f);
      cyl[2 * kRows + local] = A.z[r] * A.inv_z;
    }
    // the input of layer l's weight gradient: the lane's feature of a local row
    auto x_of = [&](int l, int kb, int q) {
      return fmaxf(A.zs[l - 1][min(t0 + q, end - 1) * W + 16 * kb + j], 0.f);
    };
    // output layer
    float dz[MB * 4], dn[MB * 4];          // column and natural layout
    {
      const float* Wo = A.W[L];
      for (int i = t; i < W * 16; i += kThreads) w[(i / 16) * LDO + i % 16] = i % 16 < A.D ? Wo[(i / 16) * A.D + i % 16] : 0.f;
      float d[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) d[v] = valid && 4 * g + v < A.D ? A.de[r * kDpad + 4 * g + v] : 0.f;
      *reinterpret_cast<float4*>(zb + local * LDO + 4 * g) = make_float4(d[0], d[1], d[2], d[3]);
      __syncthreads();
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int kb = wave + 4 * i;
        if (kb < MB)
          for (int q0 = 0; q0 < nr; q0 += 4) {
            const int q = q0 + g;
            acc_o[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x_of(L, kb, q), zb[q * LDO + j], acc_o[i], 0, 0, 0);
          }
      }
      if (t < 16)
        for (int q = 0; q < nr; ++q) bias[L] += zb[q * LDO + t];
      if (live) {
        to_nat<16>(d, d);
#pragma unroll
        for (int kb = 0; kb < MB; ++kb) {
          floatx4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s = 0; s < 4; ++s)
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(w[(16 * kb + j) * LDO + 4 * s + g], d[s], c, 0, 0, 0);
#pragma unroll
          for (int v = 0; v < 4; ++v) dz[4 * kb + v] = c[v];
        }
      }
      __syncthreads();
    }
    // hidden layers, through the ReLU of each
#pragma unroll
    for (int l = L - 1; l >= 0; --l) {
      if (live) {
        float z[MB * 4];
        load_cols<W>(z, A.zs[l] + r * W, true);
#pragma unroll
        for (int q = 0; q < MB * 4; ++q) dz[q] = valid && z[q] > 0.f ? dz[q] : 0.f;
#pragma unroll
        for (int c = 0; c < MB; ++c)
          *reinterpret_cast<float4*>(zb + local * LDZ + 16 * c + 4 * g) =
              make_float4(dz[4 * c], dz[4 * c + 1], dz[4 * c + 2], dz[4 * c + 3]);
      }
      if (l > 0) {
        const float* Wl = A.W[l];
#pragma unroll 8
        for (int i = t; i < W * W; i += kThreads) w[(i / W) * LD + i % W] = Wl[i];
      }
      __syncthreads();
      if (t < W) {
#pragma unroll 8
        for (int q = 0; q < nr; ++q) bias[l] += zb[q * LDZ + t];
      }
      if (l > 0) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          const int kb = wave + 4 * i;
          if (kb < MB)
            for (int q0 = 0; q0 < nr; q0 += 4) {
              const int q = q0 + g;
              const float x = x_of(l, kb, q);
#pragma unroll
              for (int mb = 0; mb < MB; ++mb)
                acc_h[l - 1][i][mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, zb[q * LDZ + 16 * mb + j],
                                                                           acc_h[l - 1][i][mb], 0, 0, 0);
            }
        }
        if (live) {
          to_nat<W>(dn, dz);
          floatx4 c[MB];
#pragma unroll
          for (int kb = 0; kb < MB; ++kb) c[kb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s = 0; s < MB * 4; ++s)
#pragma unroll
            for (int kb = 0; kb < MB; ++kb)
              c[kb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[(16 * kb + j) * LD + 4 * s + g], dn[s], c[kb], 0, 0, 0);
#pragma unroll
          for (int kb = 0; kb < MB; ++kb)
#pragma unroll
            for (int v = 0; v < 4; ++v) dz[4 * kb + v] = c[kb][v];
        }
      } else {
#pragma unroll
        for (int u = 0; u < NIN; ++u) {
          const int o = t + u * kThreads;
          if (o < 3 * W) {
            const float* x = cyl + (o / W) * kRows;
#pragma unroll 8
            for (int q = 0; q < nr; ++q) in_acc[u] = fmaf(x[q], zb[q * LDZ + o % W], in_acc[u]);
          }
        }
      }
      __syncthreads();
    }
  }
  float* part = A.part + (int64_t)blockIdx.x * A.part_stride;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int kb = wave + 4 * i;
    if (kb >= MB) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int k = 16 * kb + 4 * g + v;
      if (j < A.D) part[A.o[L] + k * A.D + j] = acc_o[i][v];
#pragma unroll
      for (int l = 1; l < L; ++l)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) part[A.o[l] + k * W + 16 * mb + j] = acc_h[l - 1][i][mb][v];
    }
  }
#pragma unroll
  for (int u = 0; u < NIN; ++u)
    if (t + u * kThreads < 3 * W) part[A.o[0] + t + u * kThreads] = in_acc[u];
#pragma unroll
  for (int l = 0; l < L; ++l)
    if (t < W) part[A.o[l] + (l == 0 ? 3 : W) * W + t] = bias[l];
  if (t < A.D) part[A.o[L] + W * A.D + t] = bias[L];
}

// ---------------------------------------------------------------------------
// pairwise hinge loss of the embedding
// ---------------------------------------------------------------------------

// Pairs of query q (a hit of a particle with at least three hits): its
// genuine pair (q, succ[q]); fake pairs: its hard negatives (the targets of
// the training radius graph that belong to a particle and are not succ[q])
// and its random pair (q, rnd[q]) unless that is succ[q].  Pass 0 counts them
// per block; pass 1 adds the counts, writes, per pair, g = dL/de_q (its
// negative is dL/de_b) and adds the loss.
//
// A thread walks its hit's row, a chain of loads: one-wave workgroups spread
// an event's hits over the chip.
constexpr int kHingeThreads = 64;

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) v += __shfl_xor(v, s);
  return v;
}

template <int D>
__global__ __launch_bounds__(kHingeThreads) void k_hinge(HingeArgs A, int pass) {
  if (A.status[0] != 0) return;
  float n_gen = 0.f, n_fake = 0.f, loss = 0.f;
  float inv_g = 0.f, inv_f = 0.f;
  if (pass == 1) {
    // whole numbers: exact while all pairs together are at most 2^24 (262,144 hits with
    // 64 hard negatives each), rounded as any FP32 sum beyond, in a fixed order
    float cg = 0.f, cf = 0.f;
    for (int i = threadIdx.x; i < (int)gridDim.x; i += kHingeThreads) {
      cg += A.count_part[2 * i];
      cf += A.count_part[2 * i + 1];
    }
    cg = wave_sum(cg);
    cf = wave_sum(cf);
    inv_g = cg > 0.f ? 1.0f / cg : 0.f;
    inv_f = cf > 0.f ? 1.0f / cf : 0.f;
  }
  for (int64_t q = (int64_t)blockIdx.x * kHingeThreads + threadIdx.x; q < A.n; q += (int64_t)gridDim.x * kHingeThreads) {
    float eq[D], gq[D];
#pragma unroll
    for (int k = 0; k < D; ++k) {
      eq[k] = A.emb[q * A.lde + k];
      gq[k] = 0.f;
    }
    const bool query = A.query[q] != 0;
    const int sq = A.succ[q];
    auto pair = [&](int b, bool genuine, float* gout) {
      float d2 = 0.f, diff[D];
#pragma unroll
      for (int k = 0; k < D; ++k) {
        diff[k] = eq[k] - A.emb[(int64_t)b * A.lde + k];
        d2 = fmaf(diff[k], diff[k], d2);
      }
      float c = 0.f;
      if (genuine) {
        loss += A.w_gen * d2 * inv_g;
        c = 2.f * A.w_gen * inv_g;
      } else if (A.margin - d2 > 0.f) {
        loss += (A.margin - d2) * inv_f;
        c = -2.f * inv_f;
      }
#pragma unroll
      for (int k = 0; k < D; ++k) {
        const float v = c * diff[k];
        gq[k] += v;
        if (gout) gout[k] = v;
      }
    };
    // genuine
    if (query && sq >= 0) {
      n_gen += 1.f;
      if (pass == 1) pair(sq, true, A.g_gen + q * D);
    } else if (pass == 1) {
#pragma unroll
      for (int k = 0; k < D; ++k) A.g_gen[q * D + k] = 0.f;
    }
    // hard negatives: the training radius graph's row of q
    for (int64_t t = A.row_ptr[q]; t < A.row_ptr[q + 1]; ++t) {
      const int b = A.dst[t];
      const bool fake = query && A.particle[b] >= 0 && b != sq;
      if (fake) n_fake += 1.f;
      if (pass == 1) {
        if (fake) {
          pair(b, false, A.g_edge + t * D);
        } else {
#pragma unroll
          for (int k = 0; k < D; ++k) A.g_edge[t * D + k] = 0.f;
        }
      }
    }
    // random pair
    const int rb = A.rnd[q];
    const bool rfake = query && rb >= 0 && rb != sq;
    if (rfake) n_fake += 1.f;
    if (pass == 1) {
      if (rfake) {
        pair(rb, false, A.g_rnd + q * D);
      } else {
#pragma unroll
        for (int k = 0; k < D; ++k) A.g_rnd[q * D + k] = 0.f;
      }
#pragma unroll
      for (int k = 0; k < D; ++k) A.de[q * A.ldde + k] = gq[k];
    }
  }
  if (pass == 0) {
    n_gen = wave_sum(n_gen);
    n_fake = wave_sum(n_fake);
    if (threadIdx.x == 0) {
      A.count_part[2 * blockIdx.x] = n_gen;
      A.count_part[2 * blockIdx.x + 1] = n_fake;
    }
  } else {
    loss = wave_sum(loss);
    if (threadIdx.x == 0) A.loss_part[blockIdx.x] = loss;
  }
}

// the other end of every pair: de[b] -= the pair's g, over b's in-edges of the
// training graph (CSC order), its predecessor's genuine pair and the random
// pairs that picked b (given grouped by target, in order)
template <int D>
__global__ __launch_bounds__(kHingeThreads) void k_hinge_bside(HingeArgs A) {
  if (A.status[0] != 0) return;
  for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < A.n; b += (int64_t)gridDim.x * blockDim.x) {
    float s[D];
#pragma unroll
    for (int k = 0; k < D; ++k) s[k] = 0.f;
    for (int64_t q = A.col_ptr[b]; q < A.col_ptr[b + 1]; ++q) {
      const int64_t t = A.csc[q];
#pragma unroll
      for (int k = 0; k < D; ++k) s[k] += A.g_edge[t * D + k];
    }
    const int p = A.pred[b];
    if (p >= 0)
#pragma unroll
      for (int k = 0; k < D; ++k) s[k] += A.g_gen[(int64_t)p * D + k];
    for (int64_t i = A.rnd_ptr[b]; i < A.rnd_ptr[b + 1]; ++i) {
      const int q = A.rnd_src[i];
#pragma unroll
      for (int k = 0; k < D; ++k) s[k] += A.g_rnd[(int64_t)q * D + k];
    }
#pragma unroll
    for (int k = 0; k < D; ++k) A.de[b * A.ldde + k] -= s[k];
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

hipError_t launch_emb_fwd(const EmbTrain& A, int W, int L, const etx_ctx* c, hipStream_t s) {
  if (A.n == 0) return hipSuccess;
  const dim3 grid((unsigned)std::min<int64_t>((A.n + kEmbRows - 1) / kEmbRows, (int64_t)c->n_cu * 8));
  const size_t lds = sizeof(float) * ((size_t)W * W + 2 * kEmbRows * (W + 4));
  switch (W) {
    case 32: hipLaunchKernelGGL(k_emb_fwd<32>, grid, dim3(kThreads), lds, s, A, L); break;
    case 64: hipLaunchKernelGGL(k_emb_fwd<64>, grid, dim3(kThreads), lds, s, A, L); break;
    case 128: hipLaunchKernelGGL(k_emb_fwd<128>, grid, dim3(kThreads), lds, s, A, L); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

#define EMB_BWD(X)                                                                        \
  X(32, 1) X(32, 2) X(32, 3) X(32, 4) X(64, 1) X(64, 2) X(64, 3) X(64, 4) X(128, 1)       \
  X(128, 2) X(128, 3) X(128, 4)

hipError_t launch_emb_bwd(const EmbTrain& A, int W, int L, hipStream_t s) {
  if (A.n == 0) return hipSuccess;
  const dim3 grid((unsigned)net_groups(A.n));
  const size_t lds = sizeof(float) * ((size_t)W * (W + 4) + (size_t)kRows * (W + 16) + 3 * kRows);
  switch (W * 8 + L) {
#define X(W_, L_) \
  case W_ * 8 + L_: hipLaunchKernelGGL((k_emb_bwd<W_, L_>), grid, dim3(kThreads), lds, s, A); break;
    EMB_BWD(X)
#undef X
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

int hinge_blocks(int64_t n) {
  return (int)std::max<int64_t>(1, std::min<int64_t>((n + kHingeThreads - 1) / kHingeThreads, kHingeBlocks));
}

hipError_t launch_hinge(const HingeArgs& A, int D, hipStream_t s) {
  const dim3 grid((unsigned)hinge_blocks(A.n)), block(kHingeThreads);
#define L(D_)                                                    \
  hipLaunchKernelGGL((k_hinge<D_>), grid, block, 0, s, A, 0);    \
  hipLaunchKernelGGL((k_hinge<D_>), grid, block, 0, s, A, 1);    \
  hipLaunchKernelGGL((k_hinge_bside<D_>), dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>((A.n + 63) / 64, 4096))), block, 0, s, A);
  switch (D) {
    case 4: L(4); break;
    case 8: L(8); break;
    case 12: L(12); break;
    case 16: L(16); break;
    default: return hipErrorInvalidValue;
  }
#undef L
  return hipGetLastError();
}

int train_attributes(size_t max_lds) {
  int bad = train_net_attributes(max_lds);
  auto set = [&](const void* f) {
    bad |= hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)max_lds) != hipSuccess;
  };
  set(reinterpret_cast<const void*>(k_emb_fwd<128>));
#define X(W_, L_) set(reinterpret_cast<const void*>(k_emb_bwd<W_, L_>));
  EMB_BWD(X)
#undef X
  return bad;
}

}  // namespace etx
