// 3D nearest-neighbour tables for the local greedy (Sec. 3.5, Eq. 13).
//
// M_g(t) = the g tokens nearest to t, ordered by (distance, index), t itself
// included.  Distances compare as float64 squared distances formed from the
// float32 positions as (dx^2 + dy^2) + dz^2 without fused multiply-adds, so
// the order is reproducible bit for bit.  A nonnegative double's bit pattern
// orders like its value, so each distance is a 64-bit integer key.
//
// Exact brute force over all n tokens, in two kernels.
//  - knn_bound_kernel (g <= kBoundMaxG), kQ query tokens per block: every
//    thread keeps the smallest key it sees for each query; the g-th smallest
//    of those per-thread minima, rounded up to 24 bits (bisected by one wave
//    with ballots: counting each minimum's rank took a third of the kernel),
//    is an upper bound U on the g-th smallest key (g distinct tokens lie at or
//    below it).  n = 8192, g = 64: 326 -> 101 us with the ranks of the
//    collected keys taken a query per wave.  A second pass collects the keys
//    <= U, which hold every member of M_g together with all keys tied with
//    the g-th, and ranks them by (key, index).  A row whose collection
//    overflows kCap is marked with -1 in its first entry.
//  - knn_sorted_kernel (callers with scratch space, g <= kBoundMaxG): the same
//    over tokens in spatial order (cells of a 32^3 grid in Morton order, one
//    block's counting sort).  A first bound U comes from the 256 tokens around
//    the queries in that order; a chunk of 64 tokens whose bounding box lies
//    further than U from a query holds none of its neighbours (every operation
//    of the box's distance is monotone under rounding, so the test is exact),
//    and both passes visit only the other chunks.  n = 16384, g = 17: 0.46 ms
//    over all tokens, 0.10 ms so (the sort 26 us, boxes 5, tables 68).
//  - knn_radix_kernel, one row at a time per block with all n keys in LDS
//    (n <= kKnnLdsN; for larger n each pass recomputes the keys from the
//    positions, which stay in L2): an 8-bit radix select over the key's eight
//    bytes finds the g-th smallest key T and how many keys equal to T belong
//    to the answer; the tokens below T, and the first tokens equal to T in
//    index order, are collected and ranked.  It serves g > kBoundMaxG and the
//    rows the first kernel marked.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"
#include "launch.h"

namespace cp {
namespace {

constexpr int kKnnMaxN = 32768;
constexpr int kKnnLdsN = 16384;   // up to here the radix select keeps n float64 keys (128 KiB) in LDS
constexpr int kKnnMaxG = 1024;
constexpr int kKnnBlock = 256;
constexpr int kKnnWaves = kKnnBlock / 64;
constexpr int kBoundMaxG = 128;         // <= kKnnBlock: the bound needs g per-thread minima; beyond
                                        // 128 it is loose enough that rows overflow kCap
constexpr int kQ = 8;                   // query tokens per block of the bounding kernel
constexpr int kCap = 256;               // collected keys per query

__device__ __forceinline__ unsigned long long sq_dist_key(float ax, float ay, float az, float bx, float by, float bz) {
#pragma clang fp contract(off)
  const double dx = double(ax) - double(bx), dy = double(ay) - double(by), dz = double(az) - double(bz);
  return (unsigned long long)__double_as_longlong((dx * dx + dy * dy) + dz * dz);
}

// Exclusive prefix sum over the block (thread order) with the block total.
__device__ int block_exclusive_scan(int x, int* swt, int& total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int incl = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  if (lane == 63) swt[w] = incl;
  __syncthreads();
  int before = 0;
  total = 0;
#pragma unroll
  for (int q = 0; q < kKnnWaves; ++q) {
    if (q < w) before += swt[q];
    total += swt[q];
  }
  __syncthreads();
  return before + incl - x;
}

// An upper bound on the g-th smallest of the block's 256 keys of query q, from
// their high words h (~0 for none): the smallest 24-bit prefix that g of them
// do not exceed.  One wave; ~0 when fewer than g threads hold a key.
__device__ __forceinline__ unsigned long long bound_of(const unsigned* h, int g) {
  const int lane = threadIdx.x & 63;
  unsigned v[kKnnBlock / 64];
#pragma unroll
  for (int k = 0; k < kKnnBlock / 64; ++k) v[k] = h[lane + 64 * k];
  unsigned T = 0u;
  for (int bit = 31; bit >= 8; --bit) {
    const unsigned t = T | ((1u << bit) - 1u);
    int c = 0;
#pragma unroll
    for (int k = 0; k < kKnnBlock / 64; ++k) c += __popcll(__ballot(v[k] <= t));
    if (c < g) T |= 1u << bit;
  }
  return ((unsigned long long)(T | 0xffu) << 32) | 0xffffffffull;
}

// Ranks a query's mq collected keys (one wave); the first g by (key, index)
// form its row.  More than kCap, or fewer than g, are left to the radix select.
__device__ __forceinline__ void write_row(const unsigned long long* ck, const int* ci, int mq, int g,
                                          int32_t* __restrict__ row) {
  const int lane = threadIdx.x & 63;
  if (mq > kCap || mq < g) {
    if (lane == 0) row[0] = -1;
    return;
  }
  for (int a = lane; a < mq; a += 64) {
    const unsigned long long ka = ck[a];
    const int ia = ci[a];
    int rank = 0;
    for (int b = 0; b < mq; ++b) {
      const unsigned long long kb = ck[b];
      rank += kb < ka || (kb == ka && ci[b] < ia);
    }
    if (rank < g) row[rank] = ia;
  }
}

__global__ __launch_bounds__(kKnnBlock) void knn_bound_kernel(const float* __restrict__ pos, int n, int g,
                                                              int32_t* __restrict__ out) {
  __shared__ unsigned smin[kQ][kKnnBlock];            // high words of keys
  __shared__ unsigned long long ck[kQ][kCap];
  __shared__ int ci[kQ][kCap];
  __shared__ unsigned long long sU[kQ];
  __shared__ int scount[kQ];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int q0 = blockIdx.x * kQ;
  const int nq = min(kQ, n - q0);
  float qx[kQ], qy[kQ], qz[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    const int c = q0 + min(q, nq - 1);
    qx[q] = pos[3 * c];
    qy[q] = pos[3 * c + 1];
    qz[q] = pos[3 * c + 2];
  }

  // Pass 1: the high word of every thread's smallest key for each query.
  unsigned m[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) m[q] = ~0u;
  for (int j = tid; j < n; j += kKnnBlock) {
    const float px = pos[3 * j], py = pos[3 * j + 1], pz = pos[3 * j + 2];
#pragma unroll
    for (int q = 0; q < kQ; ++q)
      m[q] = min(m[q], unsigned(sq_dist_key(qx[q], qy[q], qz[q], px, py, pz) >> 32));
  }
#pragma unroll
  for (int q = 0; q < kQ; ++q) smin[q][tid] = m[q];
  if (tid < kQ) scount[tid] = 0;
  __syncthreads();

  // U_q: g of the per-thread minima lie at or below it, so g distinct tokens do.
  for (int q = w; q < kQ; q += kKnnWaves) {
    const unsigned long long u = bound_of(smin[q], g);
    if (lane == 0) sU[q] = u;
  }
  __syncthreads();

  // Pass 2: every key <= U_q.
  unsigned long long U[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) U[q] = sU[q];
  for (int j = tid; j < n; j += kKnnBlock) {
    const float px = pos[3 * j], py = pos[3 * j + 1], pz = pos[3 * j + 2];
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const unsigned long long k = sq_dist_key(qx[q], qy[q], qz[q], px, py, pz);
      if (k <= U[q]) {
        const int slot = atomicAdd(&scount[q], 1);
        if (slot < kCap) {
          ck[q][slot] = k;
          ci[q][slot] = j;
        }
      }
    }
  }
  __syncthreads();

  // Rank the collected keys, a wave per query.
  for (int q = w; q < nq; q += kKnnWaves) write_row(ck[q], ci[q], scount[q], g, out + size_t(q0 + q) * g);
}

// Row c by radix select; keys is the block's dynamic LDS: n keys (kLds
// only), then g collected keys and g indices.  Without kLds every read of a
// key recomputes it from the positions (the same float64 value).
template <bool kLds>
__device__ void knn_radix_row(const float* __restrict__ pos, int n, int g, int c, unsigned long long* keys,
                              int32_t* __restrict__ out) {
  unsigned long long* ckey = kLds ? keys + n : keys;
  int* cidx = reinterpret_cast<int*>(ckey + g);
  __shared__ unsigned int hist[256];
  __shared__ int swt[kKnnWaves];
  __shared__ unsigned long long s_prefix;
  __shared__ int s_rank;
  const int tid = threadIdx.x;
  const float qx = pos[3 * c], qy = pos[3 * c + 1], qz = pos[3 * c + 2];
  auto key = [&](int j) -> unsigned long long {
    return kLds ? keys[j] : sq_dist_key(qx, qy, qz, pos[3 * j], pos[3 * j + 1], pos[3 * j + 2]);
  };
  if (kLds)
    for (int j = tid; j < n; j += kKnnBlock)
      keys[j] = sq_dist_key(qx, qy, qz, pos[3 * j], pos[3 * j + 1], pos[3 * j + 2]);
  if (tid == 0) {
    s_prefix = 0ull;
    s_rank = g - 1;                                     // 0-based rank of the g-th smallest
  }
  __syncthreads();

  // Radix select, most significant byte first, over the keys that share the
  // bytes chosen so far.
  unsigned long long mask = 0ull;
  for (int shift = 56; shift >= 0; shift -= 8) {
    hist[tid] = 0u;
    __syncthreads();
    const unsigned long long prefix = s_prefix;
    for (int j = tid; j < n; j += kKnnBlock) {
      const unsigned long long k = key(j);
      if ((k & mask) == prefix) atomicAdd(&hist[(k >> shift) & 255u], 1u);
    }
    __syncthreads();
    // The bucket holding rank r: its exclusive prefix count is <= r and its
    // inclusive count exceeds r.
    const int r = s_rank;
    const int h = int(hist[tid]);
    int total;
    const int before = block_exclusive_scan(h, swt, total);
    if (before <= r && r < before + h) {
      s_rank = r - before;
      s_prefix = prefix | ((unsigned long long)tid << shift);
    }
    mask |= 255ull << shift;
    __syncthreads();
  }
  const unsigned long long T = s_prefix;
  const int take_eq = s_rank + 1;                       // keys equal to T that belong to the answer

  // Collect in index order: thread tid scans the contiguous range of indices
  // [tid * span, (tid + 1) * span).
  const int span = (n + kKnnBlock - 1) / kKnnBlock;
  const int j0 = min(n, tid * span), j1 = min(n, j0 + span);
  int n_less = 0, n_eq = 0;
  for (int j = j0; j < j1; ++j) {
    const unsigned long long k = key(j);
    n_less += k < T;
    n_eq += k == T;
  }
  int less_total, eq_total;
  const int less_before = block_exclusive_scan(n_less, swt, less_total);
  const int eq_before = block_exclusive_scan(n_eq, swt, eq_total);
  (void)eq_total;
  int o_less = less_before, o_eq = eq_before;
  for (int j = j0; j < j1; ++j) {
    const unsigned long long k = key(j);
    if (k < T) {
      ckey[o_less] = k;
      cidx[o_less] = j;
      ++o_less;
    } else if (k == T) {
      if (o_eq < take_eq) {
        ckey[less_total + o_eq] = k;
        cidx[less_total + o_eq] = j;
      }
      ++o_eq;
    }
  }
  __syncthreads();

  // Place each collected pair by counting the pairs that precede it.
  for (int a = tid; a < g; a += kKnnBlock) {
    const unsigned long long ka = ckey[a];
    const int ia = cidx[a];
    int rank = 0;
    for (int b = 0; b < g; ++b) {
      const unsigned long long kb = ckey[b];
      rank += kb < ka || (kb == ka && cidx[b] < ia);
    }
    out[size_t(c) * g + rank] = ia;
  }
  __syncthreads();
}

// Rows handled by the radix select: every row (marked_only == 0) or the rows
// whose first entry the bounding kernel set to -1.  Block b takes rows
// b, b + gridDim.x, ...; it checks kKnnBlock of them at a time and selects the
// ones it must redo one after another.
template <bool kLds>
__global__ __launch_bounds__(kKnnBlock) void knn_radix_kernel(const float* __restrict__ pos, int n, int g,
                                                              int marked_only, int32_t* __restrict__ out) {
  extern __shared__ unsigned long long keys[];
  __shared__ int rows[kKnnBlock];
  __shared__ int nrows;
  const int tid = threadIdx.x;
  const int stride = gridDim.x;
  for (int base = blockIdx.x; base < n; base += stride * kKnnBlock) {
    if (tid == 0) nrows = 0;
    __syncthreads();
    const int c = base + stride * tid;
    if (c < n && (!marked_only || out[size_t(c) * g] == -1)) rows[atomicAdd(&nrows, 1)] = c;
    __syncthreads();
    const int cnt = nrows;
    for (int r = 0; r < cnt; ++r) knn_radix_row<kLds>(pos, n, g, rows[r], keys, out);
    __syncthreads();
  }
}

// Tokens in the order of their cells (order within a cell as it comes: the
// tables do not depend on it), one block.  32 cells along the longest axis.
constexpr int kSortBlock = 1024;
constexpr int kCells = 1 << 15;
constexpr int kSortU = 8;             // loads in flight
// A word of padding after every 32 cells: the threads' consecutive cells then
// start in different banks (without it the prefix took 27 us, all lanes in one).
__device__ __forceinline__ int cell_at(int c) { return c + (c >> 5); }
constexpr size_t kCellBytes = size_t(kCells + kCells / 32) * sizeof(unsigned);

__device__ __forceinline__ int cell_of(float x, float y, float z, const float* lo, float scale) {
  int code = 0;
  const float p[3] = {x, y, z};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int c = int(fminf(fmaxf((p[a] - lo[a]) * scale, 0.f), 31.f));   // fmaxf takes a NaN to 0
#pragma unroll
    for (int b = 0; b < 5; ++b) code |= ((c >> b) & 1) << (3 * b + a);
  }
  return code;
}

__global__ __launch_bounds__(kSortBlock) void knn_sort_kernel(const float* __restrict__ pos, int n,
                                                              float4* __restrict__ spos) {
  extern __shared__ unsigned cells[];                 // [kCells] counts, then each cell's next place
  __shared__ float slo[3], shi[3];
  __shared__ float wlo[kSortBlock / 64][3], whi[kSortBlock / 64][3];
  __shared__ unsigned wsum[kSortBlock / 64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  for (int i = tid; i < kCells + kCells / 32; i += kSortBlock) cells[i] = 0u;
  float lo[3], hi[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    lo[a] = __builtin_inff();
    hi[a] = -__builtin_inff();
  }
  auto each = [&](auto f) {
    for (int j0 = tid; j0 < n; j0 += kSortBlock * kSortU) {
      float p[kSortU][3];
#pragma unroll
      for (int u = 0; u < kSortU; ++u)
#pragma unroll
        for (int a = 0; a < 3; ++a) p[u][a] = pos[3 * min(j0 + u * kSortBlock, n - 1) + a];
#pragma unroll
      for (int u = 0; u < kSortU; ++u)
        if (j0 + u * kSortBlock < n) f(j0 + u * kSortBlock, p[u]);
    }
  };
  each([&](int, const float* p) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      lo[a] = fminf(lo[a], p[a]);
      hi[a] = fmaxf(hi[a], p[a]);
    }
  });
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float h = wave_max(hi[a]), l = -wave_max(-lo[a]);
    if (lane == 0) {
      wlo[w][a] = l;
      whi[w][a] = h;
    }
  }
  __syncthreads();
  if (tid < 3) {
    float l = wlo[0][tid], h = whi[0][tid];
    for (int q = 1; q < kSortBlock / 64; ++q) {
      l = fminf(l, wlo[q][tid]);
      h = fmaxf(h, whi[q][tid]);
    }
    slo[tid] = l;
    shi[tid] = h;
  }
  __syncthreads();
  const float span = fmaxf(fmaxf(shi[0] - slo[0], shi[1] - slo[1]), shi[2] - slo[2]);
  const float scale = span > 0.f ? 32.f / span : 0.f;
  each([&](int, const float* p) { atomicAdd(&cells[cell_at(cell_of(p[0], p[1], p[2], slo, scale))], 1u); });
  __syncthreads();
  // Exclusive prefix over the cells, kCells / kSortBlock consecutive ones a thread.
  constexpr int kPer = kCells / kSortBlock;
  unsigned sum = 0;
  for (int i = 0; i < kPer; ++i) sum += cells[cell_at(tid * kPer + i)];
  unsigned incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  unsigned run = incl - sum;
  for (int q = 0; q < w; ++q) run += wsum[q];
  for (int i = 0; i < kPer; ++i) {
    const unsigned c = cells[cell_at(tid * kPer + i)];
    cells[cell_at(tid * kPer + i)] = run;
    run += c;
  }
  __syncthreads();
  each([&](int j, const float* p) {
    const unsigned at = atomicAdd(&cells[cell_at(cell_of(p[0], p[1], p[2], slo, scale))], 1u);
    if (at < unsigned(n)) spos[at] = float4{p[0], p[1], p[2], __int_as_float(j)};
  });
}

// Bounding boxes of chunks of 64 tokens (one wave each).
constexpr int kChunkTokens = 64;
struct Box {
  float lo[3], hi[3];
};
__global__ __launch_bounds__(256) void knn_boxes_kernel(const float4* __restrict__ spos, int n, Box* __restrict__ box) {
  const int c = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (c * kChunkTokens >= n) return;
  const float4 p = spos[min(c * kChunkTokens + lane, n - 1)];
  // A token with a NaN is at no ordered distance: its chunk must not be ruled
  // out by the others' box, so the box takes the NaN and every test with it fails.
  const bool nan = !(p.x == p.x && p.y == p.y && p.z == p.z);
  const float v[3] = {p.x, p.y, p.z};
  const bool any = __ballot(nan) != 0ull;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float h = wave_max(v[a]), l = -wave_max(-v[a]);
    if (lane == 0) {
      box[c].lo[a] = any ? __builtin_nanf("") : l;
      box[c].hi[a] = any ? __builtin_nanf("") : h;
    }
  }
}

// The squared distance from a point to a box, formed like sq_dist_key: each
// axis' difference is 0 inside and the difference to the nearer side outside,
// so no token of the box has a smaller key.
__device__ __forceinline__ double box_dist(float x, float y, float z, const Box& b) {
#pragma clang fp contract(off)
  const float p[3] = {x, y, z};
  double d[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double below = double(b.lo[a]) - double(p[a]), above = double(p[a]) - double(b.hi[a]);
    d[a] = below > 0.0 ? below : above > 0.0 ? above : below != below ? below : 0.0;
  }
  return (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2];
}

constexpr int kMaxChunks = kKnnMaxN / kChunkTokens;

__global__ __launch_bounds__(kKnnBlock) void knn_sorted_kernel(const float4* __restrict__ spos,
                                                               const Box* __restrict__ box, int n, int g,
                                                               int32_t* __restrict__ out) {
  __shared__ unsigned smin[kQ][kKnnBlock];            // high words of keys
  __shared__ unsigned long long ck[kQ][kCap];
  __shared__ int ci[kQ][kCap];
  __shared__ unsigned long long sU[kQ];
  __shared__ int scount[kQ];
  __shared__ unsigned slist[kMaxChunks];              // chunk | queries << 16
  __shared__ int slen;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int q0 = blockIdx.x * kQ;
  const int nq = min(kQ, n - q0);
  float qx[kQ], qy[kQ], qz[kQ];
  int qt[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    const float4 p = spos[q0 + min(q, nq - 1)];
    qx[q] = p.x;
    qy[q] = p.y;
    qz[q] = p.z;
    qt[q] = __float_as_int(p.w);
  }
  // The tokens around the queries.
  {
    const int j = max(0, min(q0 + kQ / 2 - kKnnBlock / 2, n - kKnnBlock)) + tid;
    const float4 p = spos[min(j, n - 1)];
#pragma unroll
    for (int q = 0; q < kQ; ++q)
      smin[q][tid] = j < n ? unsigned(sq_dist_key(qx[q], qy[q], qz[q], p.x, p.y, p.z) >> 32) : ~0u;
  }
  if (tid < kQ) scount[tid] = 0;
  if (tid == 0) slen = 0;
  __syncthreads();
  for (int q = w; q < kQ; q += kKnnWaves) {
    const unsigned long long u = bound_of(smin[q], g);
    if (lane == 0) sU[q] = u;
  }
  __syncthreads();
  // The chunks that may hold a neighbour, and of which queries.
  unsigned long long U[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) U[q] = sU[q];
  const int nch = (n + kChunkTokens - 1) / kChunkTokens;
  for (int c = tid; c < nch; c += kKnnBlock) {
    const Box b = box[c];
    unsigned mask = 0;
#pragma unroll
    for (int q = 0; q < kQ; ++q)
      if (!(box_dist(qx[q], qy[q], qz[q], b) > __longlong_as_double((long long)U[q]))) mask |= 1u << q;
    if (mask) slist[atomicAdd(&slen, 1)] = unsigned(c) | (mask << 16);
  }
  __syncthreads();
  const int ln = slen;
  // Pass 1 over them: every thread's smallest key for each query.
  unsigned m[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) m[q] = ~0u;
  for (int i = w; i < ln; i += kKnnWaves) {
    const unsigned e = __builtin_amdgcn_readfirstlane(slist[i]);
    const int j = int(e & 0xffffu) * kChunkTokens + lane;
    const float4 p = spos[min(j, n - 1)];
#pragma unroll
    for (int q = 0; q < kQ; ++q)
      if ((e >> (16 + q)) & 1u) {
        const unsigned k = unsigned(sq_dist_key(qx[q], qy[q], qz[q], p.x, p.y, p.z) >> 32);
        m[q] = j < n && k < m[q] ? k : m[q];
      }
  }
#pragma unroll
  for (int q = 0; q < kQ; ++q) smin[q][tid] = m[q];
  __syncthreads();
  for (int q = w; q < kQ; q += kKnnWaves) {
    const unsigned long long u = bound_of(smin[q], g);
    if (lane == 0 && u < sU[q]) sU[q] = u;
  }
  __syncthreads();
  // Pass 2: every key <= U_q.
#pragma unroll
  for (int q = 0; q < kQ; ++q) U[q] = sU[q];
  for (int i = w; i < ln; i += kKnnWaves) {
    const unsigned e = __builtin_amdgcn_readfirstlane(slist[i]);
    const int j = int(e & 0xffffu) * kChunkTokens + lane;
    const float4 p = spos[min(j, n - 1)];
#pragma unroll
    for (int q = 0; q < kQ; ++q)
      if ((e >> (16 + q)) & 1u) {
        const unsigned long long k = sq_dist_key(qx[q], qy[q], qz[q], p.x, p.y, p.z);
        if (j < n && k <= U[q]) {
          const int slot = atomicAdd(&scount[q], 1);
          if (slot < kCap) {
            ck[q][slot] = k;
            ci[q][slot] = __float_as_int(p.w);
          }
        }
      }
  }
  __syncthreads();
  // Rank the collected keys, a wave per query; the first g by (key, index)
  // form the row of the query's token.
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    if ((q & (kKnnWaves - 1)) != w || q >= nq) continue;
    write_row(ck[q], ci[q], scount[q], g, out + size_t(qt[q]) * g);
  }
}

}  // namespace

static size_t knn_lds_bytes(int n, int g) { return (n <= kKnnLdsN ? size_t(n) * 8 : 0) + size_t(g) * 12; }

// The rows that the first kernel marked (bound), or all of them.
static hipError_t launch_radix(const float* pos, int n, int g, bool bound, int32_t* out, hipStream_t stream) {
  hipError_t e;
  const size_t lds = knn_lds_bytes(n, g);
  const bool in_lds = n <= kKnnLdsN;
  const void* radix = in_lds ? reinterpret_cast<const void*>(knn_radix_kernel<true>)
                             : reinterpret_cast<const void*>(knn_radix_kernel<false>);
  if ((e = hipFuncSetAttribute(radix, hipFuncAttributeMaxDynamicSharedMemorySize, int(lds))) != hipSuccess)
    return e;
  int dev = 0, cus = 0;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
  const int grid = std::max(1, std::min(n, bound ? cus : 4 * cus));
  if (in_lds)
    knn_radix_kernel<true><<<grid, kKnnBlock, lds, stream>>>(pos, n, g, bound ? 1 : 0, out);
  else
    knn_radix_kernel<false><<<grid, kKnnBlock, lds, stream>>>(pos, n, g, bound ? 1 : 0, out);
  return hipGetLastError();
}

hipError_t launch_knn(const float* pos, int n, int g, int32_t* out, hipStream_t stream) {
  if (n < 1 || n > kKnnMaxN || g < 1 || g > n || g > kKnnMaxG) return hipErrorInvalidValue;
  const bool bound = g <= kBoundMaxG;
  if (bound) {
    knn_bound_kernel<<<(n + kQ - 1) / kQ, kKnnBlock, 0, stream>>>(pos, n, g, out);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return launch_radix(pos, n, g, bound, out, stream);
}

size_t knn_boxes_bytes(int64_t n) { return size_t((n + kChunkTokens - 1) / kChunkTokens) * sizeof(Box); }

hipError_t launch_knn_sorted(const float* pos, int n, int g, int32_t* out, float4* spos, void* boxes,
                             hipStream_t stream) {
  if (n < 1 || n > kKnnMaxN || g < 1 || g > n || g > kKnnMaxG) return hipErrorInvalidValue;
  hipError_t e;
  constexpr size_t lds = kCellBytes;
  if ((e = hipFuncSetAttribute(reinterpret_cast<const void*>(knn_sort_kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize, int(lds))) != hipSuccess)
    return e;
  knn_sort_kernel<<<1, kSortBlock, lds, stream>>>(pos, n, spos);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (g > kBoundMaxG) return launch_radix(pos, n, g, false, out, stream);
  Box* box = static_cast<Box*>(boxes);
  knn_boxes_kernel<<<(n + 4 * kChunkTokens - 1) / (4 * kChunkTokens), 256, 0, stream>>>(spos, n, box);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  knn_sorted_kernel<<<(n + kQ - 1) / kQ, kKnnBlock, 0, stream>>>(spos, box, n, g, out);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return launch_radix(pos, n, g, true, out, stream);
}

}  // namespace cp
