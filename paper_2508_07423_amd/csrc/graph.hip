// Integer and graph kernels of the hot path: input validation, plane
// bucketing, edge offsets, the CSC permutation, edge compaction after the
// score cut, and union-find components.
#include "internal.hpp"

namespace etx {

namespace {

__device__ inline void set_status(int64_t* status, int64_t code) {
  atomicCAS(reinterpret_cast<unsigned long long*>(status), 0ull, static_cast<unsigned long long>(code));
}

__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline int wave_inclusive_scan(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    int t = __shfl_up(v, d);
    if (lane >= d) v += t;
  }
  return v;
}

// Exclusive scan over a 256-thread block; returns the exclusive prefix and the
// block total.  `tmp` holds 4 ints of LDS.
__device__ inline int block_exclusive_scan(int v, int* tmp, int& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int inc = wave_inclusive_scan(v);
  if (lane == 63) tmp[wave] = inc;
  __syncthreads();
  int base = 0;
  total = 0;
  for (int w = 0; w < 4; ++w) {
    int s = tmp[w];
    if (w < wave) base += s;
    total += s;
  }
  __syncthreads();
  return base + inc - v;
}

// --------------------------------------------------------------------------
// status / validation
// --------------------------------------------------------------------------

__global__ void k_init_status(int64_t* status, float* calib, int n_calib) {
  int t = threadIdx.x;
  if (t < 2) status[t] = 0;
  if (calib && t < n_calib) calib[t] = 0.f;
}

__global__ void k_validate(int64_t n_events, int64_t n_hits, const int64_t* __restrict__ hit_off,
                           const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ z,
                           const int32_t* __restrict__ plane, int n_planes, int64_t* status) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_hits + n_events + 1; i += stride) {
    if (i < n_hits) {
      int p = plane[i];
      if (!isfinite(x[i]) || !isfinite(y[i]) || !isfinite(z[i]) || p < 0 || p >= n_planes) set_status(status, ETX_ERR_INPUT);
    } else {
      int64_t e = i - n_hits;
      if (e == n_events) {
        if (hit_off[n_events] != n_hits || hit_off[0] != 0) set_status(status, ETX_ERR_INPUT);
      } else {
        int64_t cnt = hit_off[e + 1] - hit_off[e];
        if (cnt < 0) set_status(status, ETX_ERR_INPUT);
        else if (cnt > ETX_MAX_EVENT_HITS) set_status(status, ETX_ERR_UNSUPPORTED);
      }
    }
  }
}

// --------------------------------------------------------------------------
// plane bucketing: per event, a stable counting sort of hits by plane
// --------------------------------------------------------------------------

// Every thread counts a contiguous chunk of hits per plane; the waves then scan
// the 256 counts of a plane each (four per lane) and one wave the plane totals,
// so the block meets three times, not twice per plane, and eight plane numbers
// of a chunk load together: a chain of loads and barriers is all the kernel's
// time (one 1,820-hit event 14 -> 7 us).
__global__ __launch_bounds__(256) void k_bucket(const int64_t* __restrict__ hit_off, const int32_t* __restrict__ plane,
                                                int n_planes, int32_t* __restrict__ bucket,
                                                int32_t* __restrict__ plane_off, const int64_t* status) {
  constexpr int kBatch = 8;
  extern __shared__ __align__(16) int cnt[];            // [n_planes][256]
  __shared__ int base[ETX_MAX_PLANES];
  if (status[0] != 0) return;
  const int ev = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t a = hit_off[ev];
  const int n = (int)(hit_off[ev + 1] - a);
  const int chunk = (n + 255) / 256;
  const int lo = min(n, t * chunk), hi = min(n, lo + chunk);
  for (int p = 0; p < n_planes; ++p) cnt[p * 256 + t] = 0;
  auto each = [&](auto f) {
    for (int i0 = lo; i0 < hi; i0 += kBatch) {
      int pl[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) pl[u] = i0 + u < hi ? plane[a + i0 + u] : -1;
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
        if (pl[u] >= 0) f(i0 + u, pl[u]);
    }
  };
  each([&](int, int p) { cnt[p * 256 + t] += 1; });
  __syncthreads();
  for (int p = wave; p < n_planes; p += 4) {
    int4 v = *reinterpret_cast<int4*>(cnt + p * 256 + 4 * lane);
    const int sum = v.x + v.y + v.z + v.w, inc = wave_inclusive_scan(sum);
    if (lane == 63) base[p] = inc;
    int e = inc - sum;
    const int4 c = v;
    v.x = e;
    v.y = e += c.x;
    v.z = e += c.y;
    v.w = e + c.z;
    *reinterpret_cast<int4*>(cnt + p * 256 + 4 * lane) = v;
  }
  __syncthreads();
  if (wave == 0) {
    const int tot = lane < n_planes ? base[lane] : 0, ex = wave_inclusive_scan(tot) - tot;
    int32_t* po = plane_off + (int64_t)ev * (n_planes + 1);
    if (lane < n_planes) {
      base[lane] = ex;
      po[lane] = ex;
    }
    if (lane == 0) po[n_planes] = n;
  }
  __syncthreads();
  each([&](int i, int p) { bucket[a + base[p] + cnt[p * 256 + t]++] = (int32_t)(a + i); });
}

// --------------------------------------------------------------------------
// device-wide exclusive scan of per-hit edge counts -> row_ptr
// --------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_scan_reduce(const int32_t* __restrict__ cnt, int64_t n, int64_t* __restrict__ part,
                                                     const int64_t* status) {
  if (status[0] != 0) return;
  __shared__ int64_t red[256];
  int64_t b = blockIdx.x;
  int64_t s = 0;
  for (int q = 0; q < kScanBlock / 256; ++q) {
    int64_t i = b * kScanBlock + q * 256 + threadIdx.x;
    if (i < n) s += cnt[i];
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[b] = red[0];
}

// Reports more edges than the caller's capacity or than 32-bit edge ids hold;
// returns the status code.
__device__ inline int64_t check_edges(int64_t edges, int64_t capacity, int64_t* status) {
  if (edges <= capacity && edges < 0x7fffffffLL) return ETX_OK;
  const int64_t code = edges > capacity ? ETX_ERR_CAPACITY : ETX_ERR_UNSUPPORTED;
  status[1] = edges;
  set_status(status, code);
  return code;
}

__global__ __launch_bounds__(256) void k_scan_top(int64_t* __restrict__ part, int64_t nb, int64_t* __restrict__ row_ptr,
                                                  int64_t n, int64_t capacity, int64_t* status) {
  if (status[0] != 0) return;
  __shared__ int64_t sh[256];
  int64_t carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += 256) {
    int64_t b = b0 + threadIdx.x;
    int64_t v = b < nb ? part[b] : 0;
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int d = 1; d < 256; d <<= 1) {
      int64_t t = threadIdx.x >= d ? sh[threadIdx.x - d] : 0;
      __syncthreads();
      sh[threadIdx.x] += t;
      __syncthreads();
    }
    if (b < nb) part[b] = carry + sh[threadIdx.x] - v;
    int64_t tot = sh[255];
    __syncthreads();
    carry += tot;
  }
  if (threadIdx.x == 0) {
    row_ptr[n] = carry;
    check_edges(carry, capacity, status);
  }
}

// Row offsets of the kScanBlock counts from i0 on, eight consecutive counts per
// thread of a 1024-thread workgroup, starting at `carry`, which moves past them.
constexpr int kScanThreads = 1024;
static_assert(kScanBlock == 8 * kScanThreads, "eight counts per thread");

__device__ inline void scan_counts(const int32_t* __restrict__ cnt, int64_t i0, int64_t n, int64_t* __restrict__ row_ptr,
                                   int64_t& carry, int (&tot)[kScanThreads / 64]) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t i = i0 + (int64_t)t * 8;
  int v[8] = {};
  if (i + 8 <= n) {
    const int4 a = *reinterpret_cast<const int4*>(cnt + i), b = *reinterpret_cast<const int4*>(cnt + i + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  } else if (i < n) {
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = i + u < n ? cnt[i + u] : 0;
  }
  int sum = 0;
#pragma unroll
  for (int u = 0; u < 8; ++u) sum += v[u];
  const int inc = wave_inclusive_scan(sum);
  if (lane == 63) tot[wave] = inc;
  __syncthreads();
  const int of_wave = lane < kScanThreads / 64 ? tot[lane] : 0;
  const int waves = wave_inclusive_scan(of_wave);
  int64_t at = carry + __shfl(waves - of_wave, wave) + inc - sum;
  carry += __shfl(waves, kScanThreads / 64 - 1);
  if (i + 8 <= n) {
#pragma unroll
    for (int u = 0; u < 8; u += 2) {
      longlong2 r;
      r.x = at;
      r.y = at += v[u];
      at += v[u + 1];
      *reinterpret_cast<longlong2*>(row_ptr + i + u) = r;
    }
  } else if (i < n) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (i + u < n) row_ptr[i + u] = at;
      at += v[u];
    }
  }
}

__global__ __launch_bounds__(kScanThreads) void k_scan_down(const int32_t* __restrict__ cnt, int64_t n,
                                                            const int64_t* __restrict__ part,
                                                            int64_t* __restrict__ row_ptr, const int64_t* status) {
  if (status[0] != 0) return;
  __shared__ int tot[kScanThreads / 64];
  int64_t base = part[blockIdx.x];
  scan_counts(cnt, (int64_t)blockIdx.x * kScanBlock, n, row_ptr, base, tot);
}

// The whole scan of a small batch in one launch, with the capacity check and the
// per-event edge offsets: three launches fewer.  Every workgroup adds up all
// counts, for its own start and for the check, and scans its own block; what a
// small batch pays is latency: one event 25 -> 6 us, 39,000 hits (five blocks) 17 ->
// 8, 78,000 17 -> 12; 180,000 hits take 17 in four launches and 21 in one.
constexpr int64_t kSmallScan = 16 * kScanBlock;

__global__ __launch_bounds__(kScanThreads) void k_scan_small(const int32_t* __restrict__ cnt, int64_t n,
                                                             int64_t* __restrict__ row_ptr, int64_t capacity,
                                                             const int64_t* __restrict__ hit_off, int64_t n_events,
                                                             int64_t* __restrict__ edge_off, int64_t* status) {
  __shared__ int tot[kScanThreads / 64];
  __shared__ int64_t sums[3][kScanThreads / 64];
  __shared__ int64_t bad;
  // The last workgroup reports too many edges while others may still start, so a
  // workgroup's waves can read different values here: they all go on, and agree on
  // what they read where they add up their sums.  (One workgroup alone reports after
  // all its waves have read.)
  const int64_t found = status[0];
  if (gridDim.x == 1 && found != 0) return;
  const int t = threadIdx.x, lane = t & 63;
  const int64_t i0 = (int64_t)blockIdx.x * kScanBlock, i1 = i0 + kScanBlock;
  const bool last = blockIdx.x + 1 == gridDim.x;
  int64_t before = 0, all = 0;
  if (gridDim.x > 1) {
    constexpr int kBatch = 4;
    for (int64_t q0 = (int64_t)t * 4; q0 < n; q0 += 4 * kScanThreads * kBatch) {
      int4 v[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int64_t q = q0 + u * 4 * kScanThreads;
        v[u] = make_int4(0, 0, 0, 0);
        if (q + 4 <= n) v[u] = *reinterpret_cast<const int4*>(cnt + q);
        else if (q < n) v[u] = make_int4(cnt[q], q + 1 < n ? cnt[q + 1] : 0, q + 2 < n ? cnt[q + 2] : 0, 0);
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int64_t s = (int64_t)v[u].x + v[u].y + v[u].z + v[u].w;
        all += s;
        if (q0 + u * 4 * kScanThreads < i0) before += s;
      }
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
      all += __shfl_xor(all, m);
      before += __shfl_xor(before, m);
    }
    if (lane == 0) {
      sums[0][t >> 6] = before;
      sums[1][t >> 6] = all;
      sums[2][t >> 6] = found;
    }
    __syncthreads();
    before = all = 0;
    int64_t error = 0;
#pragma unroll
    for (int w = 0; w < kScanThreads / 64; ++w) {
      before += sums[0][w];
      all += sums[1][w];
      error |= sums[2][w];
    }
    if (error != 0) return;
  }
  // more edges than fit: only the last workgroup reports it, none writes offsets
  const bool fits = gridDim.x == 1 || (all <= capacity && all < 0x7fffffffLL);
  int64_t carry = before;
  if (fits) scan_counts(cnt, i0, n, row_ptr, carry, tot);
  if (t == 0) {
    bad = !fits;
    if (gridDim.x == 1) all = carry;
    if (last) {
      row_ptr[n] = all;
      bad = check_edges(all, capacity, status);
    }
  }
  __syncthreads();
  if (!edge_off || bad) return;
  for (int64_t e = t; e <= n_events; e += kScanThreads) {
    const int64_t h = hit_off[e];
    if (h >= i0 && (h < i1 || last)) edge_off[e] = row_ptr[h];
  }
}

__global__ void k_edge_off(const int64_t* __restrict__ hit_off, int64_t n_events, const int64_t* __restrict__ row_ptr,
                           int64_t* __restrict__ edge_off, const int64_t* status) {
  if (status[0] != 0) return;
  int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e <= n_events) edge_off[e] = row_ptr[hit_off[e]];
}

// --------------------------------------------------------------------------
// CSC: edge ids ordered by (dst, src), per event
// --------------------------------------------------------------------------

// The permutation of an event is built by one workgroup, in (dst, src) order
// whichever way:
//
// - Walk (long rows, at least kCscRowWalk edges per source on average, or all rows
//   where placing is off): the rows are cut into contiguous ranges, one per wave,
//   each with its own LDS cursor per target.  The waves count their edges per target, a scan over
//   (target, range) turns the counts into cursors, and every wave walks its
//   rows in order, a row per step (the targets of a row are distinct, so its
//   lanes never share a cursor).  The chain of LDS updates of one wave is what
//   bounds it, so as many waves as the cursors leave room for: kCscWords / n,
//   at most sixteen (one wave per event before: one dense 481-hit event 82 ->
//   16 us, 20 full-size events 0.55 -> 0.17 ms, 1000 uneven dense events 2.5 ->
//   1.4 ms; 1000 full-size events 1.46 -> 1.41 ms, bound by scattered 4-byte
//   writes).
// - Place (short rows): every thread drops edges into their columns through
//   LDS cursors, any order within a column, then every column is sorted by edge
//   index, which is source order (10,000 uneven events of a trained network 1.11
//   -> 0.66 ms with the wide kernel for the events of over 4,096 hits).
//
// Events of few rows and edges in a batch with more events than the chip holds
// are placed by small workgroups in memory, with an insertion sort of every column, or
// walked by them (k_csc_small); all others by
// 1024-thread workgroups with kCscWords of LDS (k_csc_wide), which place in LDS,
// as many columns at a time as fit beside the cursors, and rank every edge within
// its column instead of sorting columns (a column of sixty is then sixty short
// loops, not one long one); an event with a column too long for that walks.  Both
// kernels are launched, each skips the other's events; a batch of few events (at
// most one per CU) takes the wide kernel alone, since it then waits for the
// latency of one event.
constexpr int kCscRowWalk = 16;
// Walked events of over 2,048 hits (fewer than sixteen ranges) and fewer edges per
// hit than this take 64 edges per step, not a row: a row step is about a quarter
// microsecond, a step of 64 edges two.  300 events of 8,192 and of 16,384 hits, 1.8
// edges per hit, 0.93 -> 0.28 and 3.60 -> 1.00 ms; one of 16,384 with 5.4 edges per
// hit 1.92 by rows and 1.39 so, but 4,096 hits 0.131 and 0.126, 2,000 hits 0.042 and
// 0.060: shorter ranges than that have too few steps.
constexpr int kCscChunkRow = 4;

// The per-event kernels that keep one LDS word per hit of the event run as
// two launches: events of up to kSmallEventHits hits in workgroups with 16 KiB
// of LDS (six to eight to a CU, registers deciding, so that their chains of
// loads and barriers overlap),
// the larger ones with room for ETX_MAX_EVENT_HITS; each launch skips the
// other's events.
constexpr int kSmallEventHits = 4096;

template <int CAP>
__device__ inline bool event_in_launch(int n) {
  return CAP == kSmallEventHits ? n <= kSmallEventHits : n > kSmallEventHits;
}

// Events that k_csc_small takes.
// place: sorting a column in memory is slower than the wide workgroups' rank in LDS
// from about six edges per column on: 800 events of 490 hits, 12 edges per hit,
// 0.166 ms in memory, 0.065 in LDS; 300 of 500 hits, 4.8 per hit, 0.027 and 0.028.
// walk: events whose few edges leave sixteen waves little to do, in batches of such
// (kCscFewHits): 4,000 of 490 hits, 2 edges per hit, 0.195 ms in wide workgroups, one to
// a CU, 0.102 in small ones; of 700 hits 0.31 and 0.18.
constexpr int kCscSortRow = 6;
constexpr int kCscFewHits = 1024;                 // hits per event on average
__device__ inline bool csc_small(int n, int64_t edges, int place) {
  return place ? n <= kSmallEventHits && edges < (int64_t)kCscSortRow * n
               : n <= kCscFewHits && edges < (int64_t)kCscChunkRow * n;
}

constexpr int kCscThreads = 1024, kCscWaves = kCscThreads / 64;
constexpr int kCscWords = 32768;                  // 128 KiB: two cursors per hit of the largest event
static_assert(kCscWords >= 2 * ETX_MAX_EVENT_HITS, "two ranges of the largest event");
// Batches of small events take half: as many ranges for an event of up to 1,024
// hits, one of the largest.  Their workgroups, most of them without work, need not
// wait for a CU whose whole LDS is free behind the kernels of a batch on another
// stream (6,489 events of a trained network, two batches in turn 7.32 -> 7.02 ms
// each).
constexpr int kCscFewWords = 16384;
static_assert(kCscFewWords >= ETX_MAX_EVENT_HITS, "one range of the largest event");
static_assert(kCscFewWords >= kCscWaves * kCscFewHits, "every wave a range");

struct CscEvent {
  int64_t a, eb, ee;                              // first hit; edges
  int n;                                          // hits
  const int64_t* row_ptr;
  const int32_t* dst;
  int64_t* col_ptr;
  int32_t* csc;
};

// Counts of m columns (from hit `first` on) in R ranges -> cursors: an exclusive
// scan over columns and the ranges of each, from `base` on, which moves past them.
// T threads.  Writes the columns' starts; returns the thread's longest column.
template <int T>
__device__ inline int csc_scan(const CscEvent& E, int* cur, int first, int m, int R, int& base,
                               int (&tot)[2][T / 64]) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int slot = 0, most = 0;
  for (int i0 = 0; i0 < m; i0 += T, slot ^= 1) {
    const int i = i0 + t;
    int sum = 0;
    if (i < m)
      for (int w = 0; w < R; ++w) sum += cur[w * m + i];
    most = max(most, sum);
    const int inc = wave_inclusive_scan(sum);
    if (lane == 63) tot[slot][wave] = inc;
    __syncthreads();
    int at = base + inc - sum;
#pragma unroll
    for (int w = 0; w < T / 64; ++w) {
      at += w < wave ? tot[slot][w] : 0;
      base += tot[slot][w];
    }
    if (i < m) {
      E.col_ptr[E.a + first + i] = E.eb + at;
      for (int w = 0; w < R; ++w) {
        const int c = cur[w * m + i];
        cur[w * m + i] = at;
        at += c;
      }
    }
  }
  return most;
}

// Place: as many columns at a time as half the LDS holds cursors for (all of an
// event's, or in half the LDS those of 8,192 hits), so that the other half is left
// for their edges whatever the event's size.  With cursors for all columns an
// event of 16,384 hits had no room and walked in one range: 300 small sparse
// events and one such, 3.6 edges per hit, 3.54 ms, now 0.47 (1.5 edges per hit
// 3.34 and 0.11).  False when a column's edges do not fit.
__device__ inline bool csc_place_wide(const CscEvent& E, int* cur, int words, int (&tot)[2][kCscWaves], int& longest) {
  const int t = threadIdx.x;
  const int cols = min(E.n, words / 2), room = words - cols;
  int* list = cur + cols;
  int base = 0;
  for (int first = 0; first < E.n; first += cols) {
    const int m = min(cols, E.n - first), h0 = (int)E.a + first;
    for (int i = t; i < m; i += kCscThreads) cur[i] = 0;
    if (t == 0) longest = 0;
    __syncthreads();
    for (int64_t q = E.eb + t; q < E.ee; q += kCscThreads) {
      const int d = E.dst[q] - h0;
      if (d >= 0 && d < m) atomicAdd(&cur[d], 1);
    }
    __syncthreads();
    const int most = csc_scan<kCscThreads>(E, cur, first, m, 1, base, tot);
    if (room < E.n) atomicMax(&longest, most);
    __syncthreads();
    if (longest > room) return false;
    // cursor i is the start of column i until its edges are placed, its end
    // afterwards; as many columns at a time as their edges fit beside the cursors
    for (int lo = 0; lo < m;) {
      const int begin = cur[lo];
      int hi = m;
      if (base - begin > room) {
        int x = lo + 1;                           // the last i with cur[i] <= begin + room
        for (int step = m - x; x < hi - 1; step = (hi - x) / 2) {
          const int k = min(hi - 1, x + max(1, step));
          if (cur[k] - begin <= room) x = k;
          else hi = k;
        }
        hi = x;
      }
      const int end = hi < m ? cur[hi] : base;
      __syncthreads();                            // every thread has read the starts
      for (int64_t q = E.eb + t; q < E.ee; q += kCscThreads) {
        const int d = E.dst[q] - h0;
        if (d >= lo && d < hi) list[atomicAdd(&cur[d], 1) - begin] = (int)(q - E.eb);
      }
      __syncthreads();
      // an edge's place is the number of smaller ones in its column
      for (int j = t; j < end - begin; j += kCscThreads) {
        const int e = list[j], d = E.dst[E.eb + e] - h0;
        const int c0 = (d > lo ? cur[d - 1] : begin) - begin, c1 = cur[d] - begin;
        int rank = 0;
        for (int k = c0; k < c1; ++k) rank += list[k] < e ? 1 : 0;
        E.csc[E.eb + begin + c0 + rank] = (int32_t)(E.eb + e);
      }
      __syncthreads();
      lo = hi;
    }
  }
  return true;
}

// T threads per workgroup
template <int T>
__device__ inline void csc_walk(const CscEvent& E, int* cur, int words, int (&tot)[2][T / 64]) {
  const int t = threadIdx.x, lane = t & 63, n = E.n;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int R = min(T / 64, words / n);
  const int per = (n + R - 1) / R;                // rows per range
  const int r0 = min(n, wave * per), r1 = min(n, r0 + per);
  int* c = cur + wave * n;
  for (int i = t; i < R * n; i += T) cur[i] = 0;
  __syncthreads();
  // counts per (range, target)
  if (wave < R) {
    const int64_t q1 = E.row_ptr[E.a + r1];
    constexpr int kBatch = 8;
    for (int64_t q = E.row_ptr[E.a + r0] + lane; q < q1; q += 64 * kBatch) {
      int d[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) d[u] = q + 64 * u < q1 ? E.dst[q + 64 * u] - (int)E.a : -1;
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
        if (d[u] >= 0) atomicAdd(&c[d[u]], 1);
    }
  }
  __syncthreads();
  int base = 0;
  csc_scan<T>(E, cur, 0, n, R, base, tot);
  __syncthreads();
  if (wave >= R) return;
  if (R < T / 64 && E.ee - E.eb < (int64_t)kCscChunkRow * n) {
    // Very short rows in long ranges, 64 edges per step whatever rows they are of:
    // a lane's rank among the lanes with the same target (lower lanes are earlier
    // edges) gives its slot after the target's cursor, and the last of them moves
    // the cursor.  The next step's targets load meanwhile.  (Unrolled whole, the
    // loop's code alone made the other paths slower: one dense event 17.0 -> 18.1 us.)
    const int64_t q0 = E.row_ptr[E.a + r0], q1 = E.row_ptr[E.a + r1];
    int next = q0 + lane < q1 ? E.dst[q0 + lane] - (int)E.a : -1;
    for (int64_t q = q0 + lane; q - lane < q1; q += 64) {
      const int d = next;
      next = q + 64 < q1 ? E.dst[q + 64] - (int)E.a : -1;
      int rank = 0, count = 0;
#pragma unroll 8
      for (int k = 0; k < 64; ++k) {
        const bool same = __builtin_amdgcn_readlane(d, k) == d;
        count += same ? 1 : 0;
        rank += same && k < lane ? 1 : 0;
      }
      const int pos = d >= 0 ? c[d] + rank : 0;
      wave_sync();
      if (d >= 0) {
        E.csc[E.eb + pos] = (int32_t)q;
        if (rank == count - 1) c[d] = pos + 1;
      }
      wave_sync();
    }
    return;
  }
  // Row bounds and targets are loaded kRow rows ahead so that their latency
  // overlaps the LDS updates.
  constexpr int kRow = 8;
  int64_t rb[kRow + 1];
  int dd[kRow];
  auto load_block = [&](int i0, int64_t (&b)[kRow + 1], int (&d)[kRow]) {
#pragma unroll
    for (int q = 0; q <= kRow; ++q) b[q] = E.row_ptr[E.a + min(i0 + q, r1)];
#pragma unroll
    for (int q = 0; q < kRow; ++q) d[q] = (b[q] + lane < b[q + 1]) ? E.dst[b[q] + lane] : 0;
  };
  if (r0 < r1) load_block(r0, rb, dd);
  for (int i0 = r0; i0 < r1; i0 += kRow) {
    int64_t nb[kRow + 1];
    int nd[kRow];
    if (i0 + kRow < r1) load_block(i0 + kRow, nb, nd);
#pragma unroll
    for (int q = 0; q < kRow; ++q) {
      if (rb[q] + lane < rb[q + 1]) {
        const int dl = dd[q] - (int)E.a;
        const int pos = c[dl];
        c[dl] = pos + 1;
        E.csc[E.eb + pos] = (int32_t)(rb[q] + lane);
      }
      wave_sync();
    }
    if (i0 + kRow < r1) {
#pragma unroll
      for (int q = 0; q <= kRow; ++q) rb[q] = nb[q];
#pragma unroll
      for (int q = 0; q < kRow; ++q) dd[q] = nd[q];
    }
  }
}

__global__ __launch_bounds__(256) void k_csc_small(const int64_t* __restrict__ hit_off,
                                                   const int64_t* __restrict__ row_ptr,
                                                   const int32_t* __restrict__ dst, int64_t* __restrict__ col_ptr,
                                                   int32_t* __restrict__ csc, int place, const int64_t* status) {
  if (status[0] != 0) return;
  __shared__ int cur[kSmallEventHits];
  __shared__ int tmp[4], tot[2][4];
  const int ev = blockIdx.x, t = threadIdx.x;
  const int64_t a = hit_off[ev];
  const int n = (int)(hit_off[ev + 1] - a);
  const int64_t eb = row_ptr[a], ee = row_ptr[a + n];
  if (!csc_small(n, ee - eb, place)) return;
  if (!place) {
    if (t == 0) col_ptr[a + n] = ee;
    csc_walk<256>(CscEvent{a, eb, ee, n, row_ptr, dst, col_ptr, csc}, cur, kSmallEventHits, tot);
    return;
  }
  for (int i = t; i < n; i += 256) cur[i] = 0;
  __syncthreads();
  for (int64_t q = eb + t; q < ee; q += 256) atomicAdd(&cur[dst[q] - a], 1);
  __syncthreads();
  int base = 0;
  for (int i0 = 0; i0 < n; i0 += 256) {
    int i = i0 + t;
    int v = i < n ? cur[i] : 0;
    int total;
    int ex = block_exclusive_scan(v, tmp, total);
    if (i < n) {
      cur[i] = base + ex;
      col_ptr[a + i] = eb + base + ex;
    }
    base += total;
  }
  if (t == 0) col_ptr[a + n] = ee;
  __syncthreads();
  for (int64_t q = eb + t; q < ee; q += 256) {
    const int pos = atomicAdd(&cur[dst[q] - (int)a], 1);
    csc[eb + pos] = (int32_t)q;
  }
  __syncthreads();
  for (int i = t; i < n; i += 256) {
    const int64_t c0 = col_ptr[a + i], c1 = col_ptr[a + i + 1];
    for (int64_t j = c0 + 1; j < c1; ++j) {
      const int32_t v = csc[j];
      int64_t k = j - 1;
      for (; k >= c0; --k) {
        const int32_t u = csc[k];
        if (u < v) break;
        csc[k + 1] = u;
      }
      csc[k + 1] = v;
    }
  }
}

// place: short rows may be placed; every_event: the small kernel is not launched
__global__ __launch_bounds__(kCscThreads) void k_csc_wide(const int64_t* __restrict__ hit_off,
                                                          const int64_t* __restrict__ row_ptr,
                                                          const int32_t* __restrict__ dst,
                                                          int64_t* __restrict__ col_ptr, int32_t* __restrict__ csc,
                                                          int place, int every_event, int words,
                                                          const int64_t* status) {
  extern __shared__ int cur[];                    // cursors, and the placed edges
  __shared__ int tot[2][kCscWaves], longest;
  if (status[0] != 0) return;
  const int ev = blockIdx.x;
  const int64_t a = hit_off[ev];
  const int n = (int)(hit_off[ev + 1] - a);
  const CscEvent E{a, row_ptr[a], row_ptr[a + n], n, row_ptr, dst, col_ptr, csc};
  const int64_t edges = E.ee - E.eb;
  if (!every_event && csc_small(n, edges, place)) return;
  if (threadIdx.x == 0) col_ptr[a + n] = E.ee;
  if (n == 0) return;
  if (place && edges < (int64_t)kCscRowWalk * n && csc_place_wide(E, cur, words, tot, longest)) return;
  csc_walk<kCscThreads>(E, cur, words, tot);
}

// --------------------------------------------------------------------------
// score cut + compaction (wave ballot + block prefix scan), per event
// --------------------------------------------------------------------------

// One 1024-thread workgroup per event; every wave takes 256 consecutive scores
// per round (four ballots of 64), so a round covers 4096 edges with one
// barrier: the wave totals go to LDS (two slots, alternating between rounds,
// so that no wave overwrites a slot another wave still reads), each wave adds
// the totals of the waves before it, and every kept edge is written at its
// rank.  The kept list is in edge order.
constexpr int kCompactThreads = 1024;
constexpr int kCompactWaves = kCompactThreads / 64;
constexpr int kCompactBallots = 4;                   // 64-score ballots per wave per round

__global__ __launch_bounds__(kCompactThreads) void k_compact(const int64_t* __restrict__ hit_off,
                                                             const int64_t* __restrict__ row_ptr,
                                                             const float* __restrict__ score, float thr,
                                                             int32_t* __restrict__ kept,
                                                             int32_t* __restrict__ kept_cnt, const int64_t* status) {
  if (status[0] != 0) return;
  __shared__ int tot[2][kCompactWaves];
  const int ev = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t eb = row_ptr[hit_off[ev]], ee = row_ptr[hit_off[ev + 1]];
  const uint64_t below = (uint64_t(1) << lane) - 1;    // lanes before this one
  int64_t cnt = 0;
  int slot = 0;
  // the next round's scores are loaded before this round's barrier
  constexpr int64_t kRound = (int64_t)kCompactBallots * kCompactThreads;
  float sc[kCompactBallots];
  auto load = [&](int64_t q0) {
#pragma unroll
    for (int j = 0; j < kCompactBallots; ++j) {
      const int64_t q = q0 + (int64_t)wave * 64 * kCompactBallots + 64 * j + lane;
      sc[j] = q < ee ? score[q] : 0.f;
    }
  };
  if (eb < ee) load(eb);
  for (int64_t q0 = eb; q0 < ee; q0 += kRound) {
    const int64_t w0 = q0 + (int64_t)wave * 64 * kCompactBallots;
    uint64_t m[kCompactBallots];
    int n = 0;
#pragma unroll
    for (int j = 0; j < kCompactBallots; ++j) {
      const int64_t q = w0 + 64 * j + lane;
      m[j] = __ballot(q < ee && sc[j] >= thr);
      n += __popcll(m[j]);
    }
    if (q0 + kRound < ee) load(q0 + kRound);
    if (lane == 0) tot[slot][wave] = n;
    __syncthreads();
    int base = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kCompactWaves; ++w) {
      const int t = tot[slot][w];
      base += w < wave ? t : 0;
      total += t;
    }
#pragma unroll
    for (int j = 0; j < kCompactBallots; ++j) {
      const int64_t q = w0 + 64 * j + lane;
      if ((m[j] >> lane) & 1) kept[eb + cnt + base + __popcll(m[j] & below)] = (int32_t)q;
      base += __popcll(m[j]);
    }
    cnt += total;
    slot ^= 1;
  }
  if (threadIdx.x == 0) kept_cnt[ev] = (int32_t)cnt;
}

// --------------------------------------------------------------------------
// components: lock-free union-find in LDS, per event
// --------------------------------------------------------------------------

__device__ inline int uf_find(volatile int* par, int x) {
  int p = par[x];
  while (p != x) {
    int gp = par[p];
    if (gp != p) par[x] = gp;   // path halving: gp is an ancestor of x
    x = p;
    p = gp;
  }
  return x;
}

__device__ inline void uf_unite(volatile int* par, int u, int v) {
  while (true) {
    u = uf_find(par, u);
    v = uf_find(par, v);
    if (u == v) return;
    if (u > v) { int t = u; u = v; v = t; }
    // hook the larger root under the smaller one, so every root is its tree's minimum
    int old = atomicCAS(const_cast<int*>(reinterpret_cast<volatile int*>(par + v)), v, u);
    if (old == v) return;
    v = old;
  }
}

// Every kept edge joins its ends.  Where most edges are kept, they are read in
// order with their scores (coalesced, kUfBatch rounds in flight); where few are,
// through the kept list, a chain of two loads but no lane waits for a neighbour
// that has nothing to join.  Measured, in ms, list / scores: 1000 full-size
// events (all kept) 0.84 / 0.45, 1000 uneven dense ones 1.57 / 0.80, 10,000
// uneven ones of a trained network (two fifths kept) 0.23 / 0.33.
// T threads per event: 1024 while the batch leaves CUs idle, 256 otherwise (one
// event 18 -> 7 us, 20 full-size events 0.56 -> 0.09 ms with the scores).
constexpr int kUfBatch = 4;

template <int CAP, int T>
__global__ __launch_bounds__(T) void k_union_find(const int64_t* __restrict__ hit_off, const int64_t* __restrict__ row_ptr,
                                                  const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                  const float* __restrict__ score, float thr,
                                                  const int32_t* __restrict__ kept, const int32_t* __restrict__ kept_cnt,
                                                  int32_t* __restrict__ labels, const int64_t* status) {
  if (status[0] != 0) return;
  __shared__ int par[CAP];
  const int ev = blockIdx.x;
  const int64_t a = hit_off[ev];
  const int n = (int)(hit_off[ev + 1] - a);
  if (!event_in_launch<CAP>(n)) return;
  const int nk = kept_cnt[ev];
  const int64_t eb = row_ptr[a], ee = row_ptr[a + n];
  for (int i = threadIdx.x; i < n; i += T) par[i] = i;
  __syncthreads();
  if ((int64_t)nk * 4 < (ee - eb) * 3) {
    for (int q = threadIdx.x; q < nk; q += T) {
      const int e = kept[eb + q];
      uf_unite(par, src[e] - (int)a, dst[e] - (int)a);
    }
  } else {
    for (int64_t q0 = eb + threadIdx.x; q0 < ee; q0 += T * kUfBatch) {
      int u[kUfBatch], v[kUfBatch];
      bool keep[kUfBatch];
#pragma unroll
      for (int k = 0; k < kUfBatch; ++k) {
        const int64_t q = q0 + T * k, r = q < ee ? q : ee - 1;
        u[k] = src[r] - (int)a;
        v[k] = dst[r] - (int)a;
        keep[k] = score[r] >= thr && q < ee;
      }
#pragma unroll
      for (int k = 0; k < kUfBatch; ++k)
        if (keep[k]) uf_unite(par, u[k], v[k]);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += T) labels[a + i] = (int32_t)(a + uf_find(par, i));
}

}  // namespace

// --------------------------------------------------------------------------
// launchers
// --------------------------------------------------------------------------

#define WS(a, off, T) reinterpret_cast<T*>((a).ws + (a).L.off)

hipError_t launch_init_status(const RunArgs& a) {
  hipLaunchKernelGGL(k_init_status, dim3(1), dim3(64), 0, a.stream, a.out.status,
                     a.calibrate ? WS(a, calib, float) : nullptr, ETX_N_CALIB);
  return hipGetLastError();
}

hipError_t launch_validate(const RunArgs& a) {
  int64_t work = a.hits.n_hits + a.hits.n_events + 1;
  int grid = (int)std::min<int64_t>((work + 255) / 256, 4096);
  hipLaunchKernelGGL(k_validate, dim3(grid), dim3(256), 0, a.stream, a.hits.n_events, a.hits.n_hits, a.hits.hit_off,
                     a.hits.x, a.hits.y, a.hits.z, a.hits.plane, a.ctx->cfg.n_planes, a.out.status);
  return hipGetLastError();
}

hipError_t launch_bucket(const RunArgs& a) {
  if (a.hits.n_events == 0) return hipSuccess;
  size_t lds = sizeof(int) * 256 * a.ctx->cfg.n_planes;
  hipLaunchKernelGGL(k_bucket, dim3((unsigned)a.hits.n_events), dim3(256), lds, a.stream, a.hits.hit_off,
                     a.hits.plane, a.ctx->cfg.n_planes, WS(a, bucket, int32_t), WS(a, plane_off, int32_t),
                     a.out.status);
  return hipGetLastError();
}

hipError_t launch_scan_counts(const RunArgs& a, bool candidates) {
  // counts (ws.cnt) -> CSR offsets: the candidate offsets of the prefilter
  // path, or the main row_ptr (+ per-event edge offsets)
  const int64_t n = a.hits.n_hits;
  const int64_t nb = a.L.n_scan_blocks;
  int64_t* part = WS(a, scan_tmp, int64_t);
  int64_t* row_ptr = candidates ? WS(a, pf_tmp, int64_t) : WS(a, row_ptr, int64_t);
  if (n <= kSmallScan) {
    hipLaunchKernelGGL(k_scan_small, dim3((unsigned)std::max<int64_t>(1, nb)), dim3(kScanThreads), 0, a.stream, WS(a, cnt, int32_t), n, row_ptr,
                       a.out.edge_capacity, a.hits.hit_off, a.hits.n_events, candidates ? nullptr : a.out.edge_off,
                       a.out.status);
    return hipGetLastError();
  }
  if (nb > 0)
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(256), 0, a.stream, WS(a, cnt, int32_t), n, part,
                       a.out.status);
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(256), 0, a.stream, part, nb, row_ptr, n, a.out.edge_capacity,
                     a.out.status);
  if (nb > 0)
    hipLaunchKernelGGL(k_scan_down, dim3((unsigned)nb), dim3(kScanThreads), 0, a.stream, WS(a, cnt, int32_t), n, part, row_ptr,
                       a.out.status);
  if (!candidates) {
    int64_t ne = a.hits.n_events + 1;
    hipLaunchKernelGGL(k_edge_off, dim3((unsigned)((ne + 255) / 256)), dim3(256), 0, a.stream, a.hits.hit_off,
                       a.hits.n_events, row_ptr, a.out.edge_off, a.out.status);
  }
  return hipGetLastError();
}

hipError_t launch_csc(const RunArgs& a) {
  if (a.hits.n_events == 0) return hipSuccess;
  const dim3 grid((unsigned)a.hits.n_events);
  const int place = a.ctx->csc_place;
  const bool many = a.hits.n_events > a.ctx->n_cu, few_hits = many && a.hits.n_hits <= kCscFewHits * a.hits.n_events;
  const bool small = place ? many : few_hits;
  if (small)
    hipLaunchKernelGGL(k_csc_small, grid, dim3(256), 0, a.stream, a.hits.hit_off, WS(a, row_ptr, int64_t), a.out.dst,
                       WS(a, col_ptr, int64_t), WS(a, csc, int32_t), place, a.out.status);
  const int words = place && few_hits ? kCscFewWords : kCscWords;
  hipLaunchKernelGGL(k_csc_wide, grid, dim3(kCscThreads), sizeof(int) * words, a.stream, a.hits.hit_off,
                     WS(a, row_ptr, int64_t), a.out.dst, WS(a, col_ptr, int64_t), WS(a, csc, int32_t), place,
                     small ? 0 : 1, words, a.out.status);
  return hipGetLastError();
}

hipError_t launch_compact(const RunArgs& a) {
  if (a.hits.n_events == 0) return hipSuccess;
  hipLaunchKernelGGL(k_compact, dim3((unsigned)a.hits.n_events), dim3(kCompactThreads), 0, a.stream, a.hits.hit_off,
                     WS(a, row_ptr, int64_t), a.out.score, a.ctx->cfg.edge_threshold, WS(a, kept, int32_t),
                     WS(a, kept_cnt, int32_t), a.out.status);
  return hipGetLastError();
}

hipError_t launch_union_find(const RunArgs& a) {
  if (a.hits.n_events == 0) return hipSuccess;
#define UF(C_, T_)                                                                                                  \
  hipLaunchKernelGGL((k_union_find<C_, T_>), dim3((unsigned)a.hits.n_events), dim3(T_), 0, a.stream, a.hits.hit_off, \
                     WS(a, row_ptr, int64_t), a.out.src, a.out.dst, a.out.score, a.ctx->cfg.edge_threshold,          \
                     WS(a, kept, int32_t), WS(a, kept_cnt, int32_t),                                                 \
                     a.out.labels, a.out.status)
  const bool few = a.hits.n_events <= a.ctx->n_cu, large = a.hits.n_hits > kSmallEventHits;
  if (few) {
    UF(kSmallEventHits, 1024);
    if (large) UF(ETX_MAX_EVENT_HITS, 1024);
  } else {
    UF(kSmallEventHits, 256);
    if (large) UF(ETX_MAX_EVENT_HITS, 256);
  }
#undef UF
  return hipGetLastError();
}

int graph_attributes(size_t max_lds) {
  int bad = 0;
  bad |= hipFuncSetAttribute(reinterpret_cast<const void*>(k_bucket), hipFuncAttributeMaxDynamicSharedMemorySize, (int)max_lds) != hipSuccess;
  bad |= hipFuncSetAttribute(reinterpret_cast<const void*>(k_csc_wide), hipFuncAttributeMaxDynamicSharedMemorySize, (int)max_lds) != hipSuccess;
  return bad;
}

}  // namespace etx
