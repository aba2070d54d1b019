// FST capacity (Sec. 3.4, Eq. 9-10).
//
// r_j = (1/n) sum_{k in N_n(j)} (a_f d_f(j,k)/M_f + a_x d_x(j,k)/M_x + a_tau d_tau(j,k)/M_tau),
// v_j = r_j / sum_l r_l (uniform when every r is 0).  N_n(j) is the n tokens
// nearest to j other than j, by (squared distance, index): the first n
// entries of j's (n+1)-nearest table with j left out.  d_f = 1 - cos clamped
// to [0, 2] (cos = 0 for a zero-norm row), d_x the Euclidean distance,
// d_tau(j, k) = ReLU(tau_j - tau_k); each M is the maximum of its term over
// the n * N scored pairs (a term whose maximum is 0 contributes 0).
//
// Kernels, in stream order:
//   knn tables with g = n + 1 (k_knn.hip)
//   (from 1024 tokens on in spatial order, which the next kernel uses too)
//   cap_pairs_kernel     one wave per token: gathers each neighbour's feature
//                        row, dot product and norms in float64 (bf16 and f32
//                        products are exact there), writes the three
//                        discrepancies and raises the maxima
//   cap_score_kernel     r_j and per-block partial sums of r in fixed order
//   cap_normalise_kernel v_j = r_j / sum r, the sum taken from the partials
//                        in the same fixed order by every block
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"
#include "launch.h"

namespace cp {
namespace {

constexpr int kCapBlock = 256;
constexpr int kCapWaves = kCapBlock / kWave;

struct CapDev {
  const void* feats;
  int n, d, g, nn;                 // tokens, feature width, table width (nn + 1), neighbours
  const float* pos;
  const int32_t* frame;
  const int32_t* table;            // [n, g]
  const float4* spos;              // [n] tokens in spatial order, or null: in index order
  double* pairs;                   // [n, nn, 3]
  unsigned long long* maxbits;     // [3] float64 bits of M_f, M_x, M_tau
  double a_f, a_x, a_t;
  double* r;                       // [n]
  double* partial;                 // [ceil(n / kCapBlock)]
  float* v;                        // [n]
};

__global__ void cap_init_kernel(unsigned long long* maxbits) {
  if (threadIdx.x < 3) maxbits[threadIdx.x] = 0ull;
}

// Sums over the wave's lanes of f_a . f_b and |f_b|^2 for kCapRows rows b at a
// time, float64, and of |f_a|^2 (the first time).  Rows are read as 16-byte
// chunks: 8 bf16 or 4 float.
constexpr int kCapRows = 4;
template <bool BF16>
__device__ __forceinline__ void chunk_values(uint4 x, double (&v)[BF16 ? 8 : 4]) {
  const unsigned int xw[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    if (BF16) {
      v[2 * h] = bf16_bits_to_float(xw[h] & 0xffffu);
      v[2 * h + 1] = bf16_bits_to_float(xw[h] >> 16);
    } else {
      v[h] = __uint_as_float(xw[h]);
    }
  }
}

template <bool BF16>
__device__ __forceinline__ void rows_dots(const void* feats, int d, int a, const int (&b)[kCapRows], bool want_aa,
                                          double (&ab)[kCapRows], double (&bb)[kCapRows], double& aa) {
  const int lane = threadIdx.x & (kWave - 1);
  constexpr int kVals = BF16 ? 8 : 4;
  const int chunks = d / kVals;
  const uint4* ra = reinterpret_cast<const uint4*>(feats) + size_t(a) * chunks;
  const uint4* rb[kCapRows];
#pragma unroll
  for (int q = 0; q < kCapRows; ++q) {
    rb[q] = reinterpret_cast<const uint4*>(feats) + size_t(b[q]) * chunks;
    ab[q] = bb[q] = 0.0;
  }
  double s_aa = 0.0;
  for (int c = lane; c < chunks; c += kWave) {
    const uint4 x = ra[c];
    uint4 y[kCapRows];
#pragma unroll
    for (int q = 0; q < kCapRows; ++q) y[q] = rb[q][c];
    double xv[kVals];
    chunk_values<BF16>(x, xv);
    if (want_aa)
#pragma unroll
      for (int h = 0; h < kVals; ++h) s_aa = fma(xv[h], xv[h], s_aa);
#pragma unroll
    for (int q = 0; q < kCapRows; ++q) {
      double yv[kVals];
      chunk_values<BF16>(y[q], yv);
#pragma unroll
      for (int h = 0; h < kVals; ++h) {
        ab[q] = fma(xv[h], yv[h], ab[q]);
        bb[q] = fma(yv[h], yv[h], bb[q]);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kCapRows; ++q) {
    ab[q] = wave_sum(ab[q]);
    bb[q] = wave_sum(bb[q]);
  }
  if (want_aa) aa = wave_sum(s_aa);
}

// One wave per token, its neighbours kCapRows at a time (their rows' loads in
// flight together, the token's own row converted once for all of them).  With
// the tokens' spatial order (spos) consecutive waves take tokens that are
// close together, and so do the blocks of one XCD (block b runs on XCD b mod
// 8), whose rows then meet in its L2: bound by the gather of n nn rows, which
// otherwise comes from the Infinity Cache (n = 16384, D = 3584, nn = 16:
// 537 us in index order, one row at a time; 209 us so, half of it the float64
// conversions and products).
template <bool BF16>
__global__ __launch_bounds__(kCapBlock) void cap_pairs_kernel(CapDev p) {
  __shared__ double smax[kCapWaves][3];
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x >> 6;
  const int per = gridDim.x / 8;                      // the grid is a multiple of 8
  const int at = (int(blockIdx.x) % 8 * per + int(blockIdx.x) / 8) * kCapWaves + w;
  double mf = 0.0, mx = 0.0, mt = 0.0;
  if (at < p.n) {
    const int j = __builtin_amdgcn_readfirstlane(p.spos ? __float_as_int(p.spos[at].w) : at);
    const float xj = p.pos[3 * j], yj = p.pos[3 * j + 1], zj = p.pos[3 * j + 2];
    const int tj = p.frame[j];
    double jj = 0.0;
    int e = 0;                                        // entries of the table taken
    const int32_t* row = p.table + size_t(j) * p.g;
    for (int q0 = 0; q0 < p.nn; q0 += kCapRows) {
      // The next neighbours, the token itself left out; the last one again
      // past the end.
      int k[kCapRows];
#pragma unroll
      for (int u = 0; u < kCapRows; ++u) {
        int t = j;
        if (q0 + u < p.nn)
          while (e < p.g && (t = __builtin_amdgcn_readfirstlane(row[e++])) == j) {
          }
        k[u] = q0 + u < p.nn ? t : u > 0 ? k[u > 0 ? u - 1 : 0] : j;
      }
      double ab[kCapRows], bb[kCapRows];
      rows_dots<BF16>(p.feats, p.d, j, k, q0 == 0, ab, bb, jj);
      const double nj = sqrt(jj);
#pragma unroll
      for (int u = 0; u < kCapRows; ++u) {
        if (q0 + u >= p.nn) break;
        const double den = nj * sqrt(bb[u]);
        const double cosv = den > 0.0 ? ab[u] / den : 0.0;
        const double df = fmin(fmax(1.0 - cosv, 0.0), 2.0);
        double dx;
        {
#pragma clang fp contract(off)
          const double ex = double(xj) - double(p.pos[3 * k[u]]), ey = double(yj) - double(p.pos[3 * k[u] + 1]),
                       ez = double(zj) - double(p.pos[3 * k[u] + 2]);
          dx = sqrt((ex * ex + ey * ey) + ez * ez);
        }
        const double dt = fmax(double(tj) - double(p.frame[k[u]]), 0.0);
        if (lane == 0) {
          double* o = p.pairs + (size_t(j) * p.nn + q0 + u) * 3;
          o[0] = df;
          o[1] = dx;
          o[2] = dt;
        }
        mf = fmax(mf, df);
        mx = fmax(mx, dx);
        mt = fmax(mt, dt);
      }
    }
  }
  if (lane == 0) {
    smax[w][0] = mf;
    smax[w][1] = mx;
    smax[w][2] = mt;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    double m = 0.0;
#pragma unroll
    for (int u = 0; u < kCapWaves; ++u) m = fmax(m, smax[u][threadIdx.x]);
    // The maxima share a line that every block would update: only if it rises.
    if (m > __longlong_as_double((long long)get(p.maxbits + threadIdx.x))) atomic_max_nonneg(p.maxbits + threadIdx.x, m);
  }
}

__global__ __launch_bounds__(kCapBlock) void cap_score_kernel(CapDev p) {
  __shared__ double red[kCapBlock];
  const int j = blockIdx.x * kCapBlock + threadIdx.x;
  const double M_f = __longlong_as_double((long long)p.maxbits[0]);
  const double M_x = __longlong_as_double((long long)p.maxbits[1]);
  const double M_t = __longlong_as_double((long long)p.maxbits[2]);
  double r = 0.0;
  if (j < p.n) {
    double s = 0.0;
    const double* o = p.pairs + size_t(j) * p.nn * 3;
    for (int q = 0; q < p.nn; ++q) {
      const double tf = M_f > 0.0 ? o[3 * q] / M_f : 0.0;
      const double tx = M_x > 0.0 ? o[3 * q + 1] / M_x : 0.0;
      const double tt = M_t > 0.0 ? o[3 * q + 2] / M_t : 0.0;
      s += (p.a_f * tf + p.a_x * tx) + p.a_t * tt;
    }
    r = s / double(p.nn);
    p.r[j] = r;
  }
  red[threadIdx.x] = r;
  __syncthreads();
  for (int h = kCapBlock / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) p.partial[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(kCapBlock) void cap_normalise_kernel(CapDev p, int nparts) {
  __shared__ double stotal;
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int b = 0; b < nparts; ++b) t += p.partial[b];
    stotal = t;
  }
  __syncthreads();
  const double total = stotal;
  const int j = blockIdx.x * kCapBlock + threadIdx.x;
  if (j < p.n) p.v[j] = total > 0.0 ? float(p.r[j] / total) : float(1.0 / double(p.n));
}

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

struct CapLayout {
  size_t table, pairs, maxbits, r, partial, spos, boxes, total;
};

CapLayout cap_layout(int64_t n, int64_t nn) {
  CapLayout L;
  size_t o = 0;
  L.table = o;
  o = align256(o + size_t(n) * size_t(nn + 1) * 4);
  L.pairs = o;
  o = align256(o + size_t(n) * size_t(nn) * 24);
  L.maxbits = o;
  o = align256(o + 3 * 8);
  L.r = o;
  o = align256(o + size_t(n) * 8);
  L.partial = o;
  o = align256(o + size_t((n + kCapBlock - 1) / kCapBlock) * 8);
  L.spos = o;
  o = align256(o + size_t(n) * sizeof(float4));
  L.boxes = o;
  o = align256(o + knn_boxes_bytes(n));
  L.total = o;
  return L;
}

// From here on the spatial order pays for its two launches (about 20 us).
constexpr int kCapSortN = 1024;

}  // namespace

size_t capacity_workspace_bytes(int64_t n, int64_t nn) { return cap_layout(n, nn).total; }
size_t capacity_min_workspace_bytes(int64_t n, int64_t nn) { return cap_layout(n, nn).spos; }

hipError_t launch_capacity(const CapacityParams& c, hipStream_t stream) {
  const CapLayout L = cap_layout(c.n, c.nn);
  char* w = static_cast<char*>(c.workspace);
  CapDev p{};
  p.feats = c.feats;
  p.n = c.n;
  p.d = c.d;
  p.g = c.nn + 1;
  p.nn = c.nn;
  p.pos = c.pos;
  p.frame = c.frame;
  p.table = reinterpret_cast<int32_t*>(w + L.table);
  p.pairs = reinterpret_cast<double*>(w + L.pairs);
  p.maxbits = reinterpret_cast<unsigned long long*>(w + L.maxbits);
  p.a_f = c.alpha_f;
  p.a_x = c.alpha_x;
  p.a_t = c.alpha_tau;
  p.r = c.score ? c.score : reinterpret_cast<double*>(w + L.r);
  p.partial = reinterpret_cast<double*>(w + L.partial);
  p.v = c.capacity;

  hipError_t e;
  cap_init_kernel<<<1, 64, 0, stream>>>(p.maxbits);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  int32_t* table = reinterpret_cast<int32_t*>(w + L.table);
  if (c.n >= kCapSortN && c.workspace_bytes >= L.total) {
    float4* spos = reinterpret_cast<float4*>(w + L.spos);
    p.spos = spos;
    e = launch_knn_sorted(c.pos, c.n, p.g, table, spos, w + L.boxes, stream);
  } else {
    e = launch_knn(c.pos, c.n, p.g, table, stream);
  }
  if (e != hipSuccess) return e;
  const int pair_blocks = (c.n + 8 * kCapWaves - 1) / (8 * kCapWaves) * 8;
  if (c.bf16)
    cap_pairs_kernel<true><<<pair_blocks, kCapBlock, 0, stream>>>(p);
  else
    cap_pairs_kernel<false><<<pair_blocks, kCapBlock, 0, stream>>>(p);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int blocks = (c.n + kCapBlock - 1) / kCapBlock;
  cap_score_kernel<<<blocks, kCapBlock, 0, stream>>>(p);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  cap_normalise_kernel<<<blocks, kCapBlock, 0, stream>>>(p, blocks);
  return hipGetLastError();
}

}  // namespace cp
