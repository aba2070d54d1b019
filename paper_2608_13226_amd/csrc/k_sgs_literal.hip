// The greedy step solved as the paper writes it (Sec. 3.5, Eq. 11-15).
//
// Step l retains S_l = {s_0 .. s_{l-1}}, each with source mass u = 1/K, and
// solves the entropic semi-relaxed transport to all targets (Eq. 12:
// P 1 = u, P^T 1 <= v) by alternating scalings P = diag(a) E diag(b),
// E_ji = exp(-C(s_i, j) / eps):
//   a_i <- u / sum_j E_ji b_j,   b_j <- min(1, v_j / t_j),  t_j = sum_i E_ji a_i
// (b_j = 1 where t_j = 0), from b = 1, for a fixed number of rounds.  The
// residual r_j = max(0, v_j - b_j t_j) (Eq. 14) weights the score
// score(c) = sum_j r_j C(c, j) (Eq. 15 with every target a neighbour), and
// the unselected token with the smallest score is retained next (ties to the
// smaller index).  Step 0 has no source and r = v.  After K picks the same
// solve over all of S gives the plan whose cost <P, C_S> is reported.
//
// Layout: E is a compact [n, kp] float64 matrix (kp = k rounded up to 4)
// whose column i is filled when s_i is retained, target-major like the
// cost, so a round is one pass over the first l columns.  Kernels, per step:
//   lit_append_kernel   E[:, l-1] = exp(-C_tm[:, s_{l-1}] / eps) in float64
//                       (float32 would flush exp(-C / eps) to zero once C / eps
//                       passes about 103, cutting sources off from targets
//                       they must reach; float64 holds it to about 708)
//   lit_rows_kernel     64 rows per block: t_j (one wave per row), b_j, and
//                       the block's column sums sum_j E_ji b_j (one thread per
//                       column); b = 1 on the first round
//   lit_a_kernel        a_i = u / (sum of the row blocks' column sums, in
//                       block order)
//   lit_rows_kernel     (last round) r_j instead of column sums
//   lit_score_kernel    row panels x 256-column strips: partial sum_j r_j C_tm[j][c]
//   lit_select_kernel   one block: panel sums in panel order, argmin over the
//                       unselected tokens, residual mass
// Every sum is float64 in a fixed order, so results are deterministic.
// Small scenes run in one persistent launch instead (lit_persistent_kernel).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>

#include "sgs_exchange.h"

namespace cp {
namespace {

constexpr int kLitBlock = 256;
constexpr int kLitWaves = kLitBlock / kWave;
constexpr int kLitRows = 64;          // rows per block of lit_rows_kernel
constexpr int kLitMaxK = 4096;        // a (float64) and the picks stay in LDS
constexpr int kSelectBlock = 1024;

struct LitDev {
  const float* C;          // [n, n] target-major
  const float* v;          // [n]
  int n, k, kp;
  double eps, u;
  double* E;               // [n, kp]
  double* a;               // [k]
  double* b;               // [n]
  double* r;               // [n]
  double* colpart;         // [kp, nrb]: column i's partial sums, one per row block
  double* scorepart;       // [panels, n]
  double* objpart;         // [nrb]
  unsigned char* chosen;   // [n]
  int32_t* selected;       // [k]
  const int32_t* follow;   // [k] or nullptr
  double* step_score;      // [k] or nullptr
  double* step_residual;   // [k] or nullptr
  double* objective;       // [1] or nullptr
  int nrb, panels, strips;
};

__global__ void lit_init_kernel(LitDev p) {
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < p.n; j += gridDim.x * blockDim.x) {
    p.chosen[j] = 0;
    p.r[j] = double(p.v[j]);
  }
}

// Column l - 1 of E from the pick of step l - 1.
__global__ void lit_append_kernel(LitDev p, int l) {
  const int s = min(max(int(p.selected[l - 1]), 0), p.n - 1);
  if (blockIdx.x == 0 && threadIdx.x == 0) p.chosen[s] = 1;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < p.n; j += gridDim.x * blockDim.x)
    p.E[size_t(j) * p.kp + (l - 1)] = exp(-double(p.C[size_t(j) * p.n + s]) / p.eps);
}

// mode 0: first round (b = 1): column sums only.
// mode 1: t_j, b_j, then column sums with the new b.
// mode 2: last round: t_j, b_j and the residual r_j.
__global__ __launch_bounds__(kLitBlock) void lit_rows_kernel(LitDev p, int l, int mode) {
  __shared__ double sa[kLitMaxK];
  __shared__ double sb[kLitRows];
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x >> 6;
  const int j0 = blockIdx.x * kLitRows;
  const int rows = min(kLitRows, p.n - j0);
  if (mode == 0) {
    for (int q = threadIdx.x; q < rows; q += kLitBlock) sb[q] = 1.0;
  } else {
    for (int i = threadIdx.x; i < l; i += kLitBlock) sa[i] = p.a[i];
    __syncthreads();
    for (int q = w; q < rows; q += kLitWaves) {
      const int j = j0 + q;
      const double* e = p.E + size_t(j) * p.kp;
      double t = 0.0;
#pragma unroll 4
      for (int i = lane; i < l; i += kWave) t = fma(e[i], sa[i], t);
      t = wave_sum(t);
      const double vj = double(p.v[j]);
      const double bj = t > 0.0 ? fmin(1.0, vj / t) : 1.0;
      if (lane == 0) {
        sb[q] = bj;
        p.b[j] = bj;
        if (mode == 2) p.r[j] = fmax(vj - bj * t, 0.0);
      }
    }
  }
  if (mode == 2) return;
  __syncthreads();
  for (int i = threadIdx.x; i < l; i += kLitBlock) {
    double s = 0.0;
#pragma unroll 8
    for (int q = 0; q < rows; ++q) s = fma(p.E[size_t(j0 + q) * p.kp + i], sb[q], s);
    p.colpart[size_t(i) * p.nrb + blockIdx.x] = s;
  }
}

// One wave per column: its row-block partials, lane-strided then a fixed
// butterfly, so the sum's order does not depend on timing.
__global__ __launch_bounds__(kLitBlock) void lit_a_kernel(LitDev p, int l) {
  const int lane = threadIdx.x & (kWave - 1);
  const int i = blockIdx.x * kLitWaves + (threadIdx.x >> 6);
  if (i >= l) return;
  const double* c = p.colpart + size_t(i) * p.nrb;
  double s = 0.0;
  for (int rb = lane; rb < p.nrb; rb += kWave) s += c[rb];
  s = wave_sum(s);
  if (lane == 0) p.a[i] = p.u / s;
}

// Partial scores: block (strip, panel) sums r_j C_tm[j][c] over the panel's
// rows for the strip's 256 columns, eight rows in flight per thread.
__global__ __launch_bounds__(kLitBlock) void lit_score_kernel(LitDev p) {
  __shared__ double sr[kLitBlock];
  const int c = blockIdx.x * kLitBlock + threadIdx.x;
  const int per = (p.n + p.panels - 1) / p.panels;
  const int r0 = blockIdx.y * per, r1 = min(p.n, r0 + per);
  double acc = 0.0;
  for (int base = r0; base < r1; base += kLitBlock) {
    const int cnt = min(kLitBlock, r1 - base);
    __syncthreads();
    if (threadIdx.x < cnt) sr[threadIdx.x] = p.r[base + threadIdx.x];
    __syncthreads();
    if (c < p.n) {
      int q = 0;
      for (; q + 8 <= cnt; q += 8) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = __builtin_nontemporal_load(p.C + size_t(base + q + u) * p.n + c);
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = fma(sr[q + u], double(x[u]), acc);
      }
      for (; q < cnt; ++q) acc = fma(sr[q], double(p.C[size_t(base + q) * p.n + c]), acc);
    }
  }
  if (c < p.n) p.scorepart[size_t(blockIdx.y) * p.n + c] = acc;
}

// Step l's pick: panel sums in panel order, the smallest score over the
// unselected tokens (smaller index on ties), and the residual mass.
__global__ __launch_bounds__(kSelectBlock) void lit_select_kernel(LitDev p, int l) {
  __shared__ double sv[kSelectBlock];
  __shared__ int si[kSelectBlock];
  __shared__ double sm[kSelectBlock];
  double best = DBL_MAX, mass = 0.0;
  int bi = INT_MAX;
  for (int c = threadIdx.x; c < p.n; c += kSelectBlock) {
    mass += p.r[c];
    if (p.chosen[c]) continue;
    double s = 0.0;
    for (int q = 0; q < p.panels; ++q) s += p.scorepart[size_t(q) * p.n + c];
    if (s < best) {
      best = s;
      bi = c;
    }
  }
  sv[threadIdx.x] = best;
  si[threadIdx.x] = bi;
  sm[threadIdx.x] = mass;
  __syncthreads();
  for (int h = kSelectBlock / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) {
      const double ov = sv[threadIdx.x + h];
      const int oi = si[threadIdx.x + h];
      if (ov < sv[threadIdx.x] || (ov == sv[threadIdx.x] && oi < si[threadIdx.x])) {
        sv[threadIdx.x] = ov;
        si[threadIdx.x] = oi;
      }
      sm[threadIdx.x] += sm[threadIdx.x + h];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    int pick = si[0];
    double score = sv[0];
    if (p.follow) {
      pick = min(max(int(p.follow[l]), 0), p.n - 1);
      score = 0.0;
      for (int q = 0; q < p.panels; ++q) score += p.scorepart[size_t(q) * p.n + pick];
    }
    p.selected[l] = pick;
    if (p.step_score) p.step_score[l] = score;
    if (p.step_residual) p.step_residual[l] = sm[0];
  }
}

// The picks of a trajectory to follow, when no per-step output is wanted.
__global__ void lit_follow_kernel(LitDev p) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < p.k; i += gridDim.x * blockDim.x)
    p.selected[i] = min(max(int(p.follow[i]), 0), p.n - 1);
}

// Transport cost of the final plan: block partials of
// sum_j sum_i a_i E_ji b_j C(s_i, j).
__global__ __launch_bounds__(kLitBlock) void lit_objective_kernel(LitDev p) {
  __shared__ double sa[kLitMaxK];
  __shared__ int ss[kLitMaxK];
  __shared__ double sw[kLitWaves];
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x >> 6;
  for (int i = threadIdx.x; i < p.k; i += kLitBlock) {
    sa[i] = p.a[i];
    ss[i] = min(max(int(p.selected[i]), 0), p.n - 1);
  }
  __syncthreads();
  const int j0 = blockIdx.x * kLitRows;
  const int rows = min(kLitRows, p.n - j0);
  double acc = 0.0;
  for (int q = w; q < rows; q += kLitWaves) {
    const int j = j0 + q;
    const double* e = p.E + size_t(j) * p.kp;
    const float* c = p.C + size_t(j) * p.n;
    double s = 0.0;
    for (int i = lane; i < p.k; i += kWave) s = fma(sa[i] * e[i], double(c[ss[i]]), s);
    acc += wave_sum(s) * p.b[j];
  }
  if (lane == 0) sw[w] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int q = 0; q < kLitWaves; ++q) s += sw[q];
    p.objpart[blockIdx.x] = s;
  }
}

__global__ void lit_objective_sum_kernel(LitDev p) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    double s = 0.0;
    for (int rb = 0; rb < p.nrb; ++rb) s += p.objpart[rb];
    *p.objective = s;
  }
}

// ---------------------------------------------------------------------------
// The same greedy in one cooperative launch, for scenes whose E fits in
// registers and whose cost in LDS (n <= kPersN, k <= kPersK, rounds <= kPersRounds; no
// trajectory to follow).
//
// A scaling round is two dependent passes over a small matrix (3.4 MB at
// n = 2048, k = 205), and 10 250 rounds follow one another: as two launches a
// round they took 18 us, nearly all of it launching and filling the pipeline.
// Here ceil(n / 64) solver blocks keep 64 rows of E each in registers (wave w
// rows 8 w .. 8 w + 7, lane and chunk the column) for the whole call.  Per
// round a solver forms t_j and b_j of its rows, its column sums, and publishes
// them; every solver then adds all blocks' sums in block order and holds the
// same a_i.  A column sum is nonnegative, so its sign bit carries the epoch of
// the exchange: one trip through memory a round, no flags and no grid barrier.
// After the last round the residuals go to the scoring blocks (ceil(n / 8),
// each with 8 rows of the cost in LDS), which write their partial scores;
// block b adds the partials of candidates 8 b .. 8 b + 7, publishes its best
// one, and every block takes the same pick.  Bound by the exchange (about
// 2 us a round) and the chain of sums, divisions and barriers around it (as
// long again); n = 2048, k = 205, 50 rounds: 177 ms as launches, 46 ms here.
constexpr int kPersN = 2048;
constexpr int kPersK = 256;
constexpr int kPersRows = 64;                         // rows of E a solver block holds
constexpr int kPersSolvers = kPersN / kPersRows;      // 32
constexpr int kPersScore = 8;                         // rows of the cost a block holds, and candidates it adds up
constexpr int kPersBlocks = kPersN / kPersScore;      // 256
constexpr int kPersChunks = kPersK / 64;              // columns a lane holds
// The scoring blocks poll through a whole solve, `rounds` exchanges of 4.4 us,
// within the limit of about a second that bounds every wait: up to this many
// rounds (72 ms) a solve stays far below it.  Longer ones take the separate
// launches, which wait for nothing.
constexpr int kPersRounds = 16384;

struct LitPers {
  const float* C;
  const float* v;
  int n, k, rounds;
  double eps, u;
  int32_t* selected;
  double* step_score;
  double* step_residual;
  double* objpart;               // [solvers]
  unsigned long long* col;       // [2][kPersSolvers][kPersK] column sums, epoch in the sign
  unsigned long long* r;         // [2][kPersN] residuals, epoch in the sign
  unsigned long long* mass;      // [2][kPersSolvers] their sums, epoch in the sign
  double* part;                  // [blocks][n] partial scores
  unsigned long long* flag;      // [kPersBlocks] slots: steps whose partial scores are written
  unsigned long long* cand;      // [2][kPersBlocks] slots: score high, score low, index, each above the step
  unsigned int* abort;
  unsigned int poll_limit, abort_init;
  int solvers;
};

__global__ void lit_pers_init_kernel(LitPers p, size_t words) {
  const size_t gt = size_t(blockIdx.x) * blockDim.x + threadIdx.x, nt = size_t(gridDim.x) * blockDim.x;
  for (size_t i = gt; i < words; i += nt) p.col[i] = 0ull;   // col, r, mass, flag and cand lie side by side
  if (gt == 0) *p.abort = p.abort_init;
}

__device__ __forceinline__ double lane_f64(double x, int l) {
  return __longlong_as_double((long long)lane_u64((unsigned long long)__double_as_longlong(x), l));
}
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  return __longlong_as_double((long long)dpp_u64<CTRL>((unsigned long long)__double_as_longlong(x)));
}

// Sums of eight values over the wave: lane l ends with the sum of value
// (l & 7).  Halving by lane bits 0 and 1, whole rotation by 8, halving by
// bit 2 (a rotation by 4 is one by lane ^ 4 once the values repeat every 8),
// then the four rows of 16.
__device__ __forceinline__ double wave_sum8(const double (&p)[8]) {
  const int lane = threadIdx.x & 63;
  double a[4], b[2];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const bool odd = lane & 1;
    a[q] = (odd ? p[2 * q + 1] : p[2 * q]) + dpp_f64<0xB1>(odd ? p[2 * q] : p[2 * q + 1]);
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const bool odd = lane & 2;
    b[q] = (odd ? a[2 * q + 1] : a[2 * q]) + dpp_f64<0x4E>(odd ? a[2 * q] : a[2 * q + 1]);
    b[q] += dpp_f64<0x128>(b[q]);
  }
  const bool odd = lane & 4;
  double x = (odd ? b[1] : b[0]) + dpp_f64<0x124>(odd ? b[0] : b[1]);
  x += __shfl_xor(x, 16);
  x += __shfl_xor(x, 32);
  return x;
}

// x with the exchange's epoch in its sign; x is not negative.
__device__ __forceinline__ unsigned long long signed_word(double x, unsigned long long epoch) {
  return ((unsigned long long)__double_as_longlong(x) & ~kEpoch) | epoch;
}
__device__ __forceinline__ double word_value(unsigned long long x) { return __longlong_as_double((long long)(x & ~kEpoch)); }

// The order of doubles as that of unsigned integers.
__device__ __forceinline__ unsigned long long f64_order(double x) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  return (b & kEpoch) ? ~b : (b | kEpoch);
}

__global__ __launch_bounds__(kBlock) void lit_persistent_kernel(LitPers p) {
  extern __shared__ float scost[];                    // [kPersScore][n] rows of the cost to score
  const int blk = blockIdx.x, nt = gridDim.x;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  __shared__ double sa[kPersK];                       // a of the round
  __shared__ double sred[kWaves][kPersK];             // the waves' column sums; scores
  __shared__ double shalf[kPersK];                    // sums over the second half of the blocks
  __shared__ double sr[kPersScore];                   // residuals of the scored rows
  __shared__ unsigned long long su[kWaves];
  __shared__ int si[kWaves];
  __shared__ int spick[kPersK];
  __shared__ int sflag;
  __shared__ double smass[kWaves];

  const bool solver = blk < p.solvers;
  // Rows of E: 8 of this wave, columns lane, lane + 64, ..; zero where there
  // is no column yet and past n.
  double E[8][kPersChunks];
#pragma unroll
  for (int q = 0; q < 8; ++q)
#pragma unroll
    for (int c = 0; c < kPersChunks; ++c) E[q][c] = 0.0;
  const int jw = blk * kPersRows + w * 8;             // the wave's first row (solvers)
  const int jl = jw + (lane & 7);                     // the lane's row
  const double vl = solver && jl < p.n ? double(p.v[jl]) : 0.0;
  for (int q = 0; q < kPersScore; ++q) {
    const int j = blk * kPersScore + q;
    for (int c = tid; c < p.n; c += kBlock) scost[q * p.n + c] = j < p.n ? p.C[size_t(j) * p.n + c] : 0.f;
  }
  unsigned chosen = 0;                                // of the candidates 8 blk .. 8 blk + 7
  if (tid == 0) sflag = 0;
  if (tid < kPersK) sa[tid] = 0.0;
  __syncthreads();

  int round = 0;                                      // exchanges of column sums so far
  double t8 = 0.0, b8 = 1.0;                          // t and b of the lane's row
  // Column sums of the own rows for the current b, all blocks' added up, and
  // the new a.  False when the launch gives up.
  auto scale_a = [&](int l) -> bool {
    const int nc = (l + 63) >> 6;
    double s[kPersChunks];
#pragma unroll
    for (int c = 0; c < kPersChunks; ++c) s[c] = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const double bq = lane_f64(b8, q);
#pragma unroll
      for (int c = 0; c < kPersChunks; ++c)
        if (c < nc) s[c] = fma(E[q][c], bq, s[c]);
    }
#pragma unroll
    for (int c = 0; c < kPersChunks; ++c)
      if (c < nc) sred[w][c * 64 + lane] = s[c];
    __syncthreads();
    const unsigned long long ep = epoch_of(round);
    unsigned long long* set = p.col + size_t(round & 1) * kPersSolvers * kPersK;
    const int i = tid & (kPersK - 1), h = tid / kPersK;     // column, half of the blocks
    // Every column's word every round, also of columns not in use yet: the
    // epoch of a word tells only this round's from the one two before.
    if (h == 0) {
      double x = 0.0;
      if (i < l)
#pragma unroll
        for (int q = 0; q < kWaves; ++q) x += sred[q][i];
      put(set + size_t(blk) * kPersK + i, signed_word(x, ep));
    }
    double sum = 0.0;
    if (i < l) {
      constexpr int kHalf = kPersSolvers / 2;
      unsigned long long x[kHalf];
#pragma unroll
      for (int q = 0; q < kHalf; ++q) x[q] = ~ep;
      for (unsigned int spins = 0;; ++spins) {
        bool miss = false;
#pragma unroll
        for (int q = 0; q < kHalf; ++q)
          if (h * kHalf + q < p.solvers && (x[q] & kEpoch) != ep) x[q] = get(set + size_t(h * kHalf + q) * kPersK + i);
#pragma unroll
        for (int q = 0; q < kHalf; ++q) miss = miss || (h * kHalf + q < p.solvers && (x[q] & kEpoch) != ep);
        if (!miss) break;
        if (give_up(spins, p.poll_limit, p.abort)) {
          sflag = 1;
          break;
        }
      }
#pragma unroll
      for (int q = 0; q < kHalf; ++q)
        if (h * kHalf + q < p.solvers) sum += word_value(x[q]);
    }
    ++round;
    if (h == 1 && i < l) shalf[i] = sum;
    __syncthreads();
    if (h == 0 && i < l) sa[i] = p.u / (sum + shalf[i]);
    __syncthreads();
    return sflag == 0;
  };
  // t and b of the own rows from a.
  auto scale_b = [&](int l) {
    const int nc = (l + 63) >> 6;
    double x[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = 0.0;
#pragma unroll
    for (int c = 0; c < kPersChunks; ++c)
      if (c < nc) {
        const double ac = sa[c * 64 + lane];
#pragma unroll
        for (int q = 0; q < 8; ++q) x[q] = fma(E[q][c], ac, x[q]);
      }
    t8 = wave_sum8(x);
    b8 = t8 > 0.0 ? fmin(1.0, vl / t8) : 1.0;
  };
  auto solve = [&](int l) -> bool {
    b8 = 1.0;
    for (int it = 0; it < p.rounds; ++it) {
      if (!scale_a(l)) return false;
      scale_b(l);
    }
    return true;
  };

  for (int l = 0; l < p.k; ++l) {
    const unsigned long long ep = epoch_of(l);
    // The residuals (step 0: the capacities) and their sum per solver.
    if (solver) {
      double res = vl;
      if (l > 0) {
        if (!solve(l)) return;
        res = fmax(vl - b8 * t8, 0.0);
      }
      if (lane < 8 && jl < p.n) put(p.r + size_t(l & 1) * kPersN + jl, signed_word(res, ep));
      double m = lane < 8 ? res : 0.0;
      m += dpp_f64<0xB1>(m);
      m += dpp_f64<0x4E>(m);
      m += __shfl_xor(m, 4);
      if (lane == 0) smass[w] = m;
      __syncthreads();
      if (tid == 0) {
        double x = 0.0;
        for (int q = 0; q < kWaves; ++q) x += smass[q];
        put(p.mass + size_t(l & 1) * kPersSolvers + blk, signed_word(x, ep));
      }
    }
    // Residuals of the rows this block scores.
    if (tid < kPersScore) {
      const int j = blk * kPersScore + tid;
      double x = 0.0;
      if (j < p.n) {
        unsigned long long y = ~ep;
        if (!wait_slot(p.r + size_t(l & 1) * kPersN + j, p.abort, p.poll_limit,
                       [ep](unsigned long long z) { return (z & kEpoch) == ep; }, y))
          sflag = 1;
        x = word_value(y);
      }
      sr[tid] = x;
    }
    __syncthreads();
    if (sflag) return;
    for (int col = tid; col < p.n; col += kBlock) {
      double x = 0.0;
#pragma unroll
      for (int q = 0; q < kPersScore; ++q) x = fma(sr[q], double(scost[q * p.n + col]), x);
      put(p.part + size_t(blk) * p.n + col, x);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);               // vmcnt(0): this wave's stores are done
    __syncthreads();
    const unsigned long long tag = (unsigned long long)(l + 1);
    if (tid == 0) put(p.flag + size_t(blk) * kSlotStride, tag);
    // Every block's partial scores of the own candidates, added in a fixed
    // order: thread (candidate, part) takes blocks part, part + 64, ...
    if (tid < nt) {
      unsigned long long y;
      if (!wait_slot(p.flag + size_t(tid) * kSlotStride, p.abort, p.poll_limit,
                     [tag](unsigned long long z) { return z >= tag; }, y))
        sflag = 1;
    }
    __syncthreads();
    if (sflag) return;
    {
      const int c = tid & (kPersScore - 1), part = tid / kPersScore;
      const int col = min(blk * kPersScore + c, p.n - 1);
      double x[kPersBlocks / 64];
#pragma unroll
      for (int q = 0; q < kPersBlocks / 64; ++q)
        x[q] = get(p.part + size_t(min(part + 64 * q, nt - 1)) * p.n + col);
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < kPersBlocks / 64; ++q)
        if (part + 64 * q < nt) s += x[q];
      // Lanes 8 apart hold one candidate: the wave's eight parts, then the waves'.
      s += dpp_f64<0x128>(s);
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      if (lane < kPersScore) sred[w][lane] = s;
    }
    __syncthreads();
    if (w == 0) {
      const int col = blk * kPersScore + lane;
      const bool ok = lane < kPersScore && col < p.n && !((chosen >> (lane & 7)) & 1u);
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < kWaves; ++q) s += sred[q][lane & 7];
      // As in lit_select_kernel a NaN (an infinite cost where nothing is left)
      // comes after every finite score, whatever its sign.
      const unsigned long long key = ok ? ~f64_order(s < DBL_MAX ? s : double(__builtin_inff())) : 0ull;
      const unsigned long long top = wave_max_u64(key);
      const int bi = wave_min_i32(ok && key == top ? col : INT_MAX);
      // The best one's score (none: no word of it is taken).
      const unsigned long long bits = ~top;
      if (lane < 3) {
        const unsigned pay = lane == 0 ? unsigned(bits >> 32) : lane == 1 ? unsigned(bits) : unsigned(bi);
        put(p.cand + (size_t(l & 1) * kPersBlocks + blk) * kSlotStride + lane, (tag << 32) | pay);
      }
    }
    // Every block's candidate; the smallest score, then the smallest index.
    {
      unsigned long long key = 0ull;
      int bi = INT_MAX;
      if (tid < nt) {
        const unsigned long long* slot = p.cand + (size_t(l & 1) * kPersBlocks + tid) * kSlotStride;
        for (unsigned int spins = 0;; ++spins) {
          const unsigned long long x0 = get(slot), x1 = get(slot + 1), x2 = get(slot + 2);
          if ((x0 >> 32) == tag && (x1 >> 32) == tag && (x2 >> 32) == tag) {
            bi = int(unsigned(x2));
            key = bi == INT_MAX ? 0ull : ~((x0 << 32) | (x1 & 0xffffffffull));
            break;
          }
          if (give_up(spins, p.poll_limit, p.abort)) {
            sflag = 1;
            break;
          }
          __builtin_amdgcn_s_sleep(1);
        }
      }
      const unsigned long long top = wave_max_u64(key);
      const int im = wave_min_i32(key == top ? bi : INT_MAX);
      if (lane == 0) {
        su[w] = top;
        si[w] = im;
      }
    }
    __syncthreads();
    if (sflag) return;
    unsigned long long top = su[0];
    int s = si[0];
#pragma unroll
    for (int q = 1; q < kWaves; ++q)
      if (su[q] > top || (su[q] == top && si[q] < s)) {
        top = su[q];
        s = si[q];
      }
    s = min(s, p.n - 1);
    if (s / kPersScore == blk) chosen |= 1u << (s % kPersScore);
    if (tid == 0) {
      spick[l] = s;
      if (blk == 0) {
        p.selected[l] = s;
        if (p.step_score) {
          const unsigned long long o = ~top;            // f64_order of the score
          p.step_score[l] = __longlong_as_double((long long)((o & kEpoch) ? (o & ~kEpoch) : ~o));
        }
      }
    }
    if (blk == 0 && w == 1 && p.step_residual) {
      double m = 0.0;
      bool ok = true;
      if (lane < p.solvers) {
        unsigned long long y = 0;
        ok = wait_slot(p.mass + size_t(l & 1) * kPersSolvers + lane, p.abort, p.poll_limit,
                       [ep](unsigned long long z) { return (z & kEpoch) == ep; }, y);
        m = word_value(y);
      }
      m = wave_sum(m);
      if (lane == 0 && ok) p.step_residual[l] = m;
    }
    // The pick's column of E.
    if (solver) {
      const double x = jl < p.n ? exp(-double(p.C[size_t(jl) * p.n + s]) / p.eps) : 0.0;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const double xq = lane_f64(x, q);
#pragma unroll
        for (int c = 0; c < kPersChunks; ++c)
          if (c == (l >> 6) && lane == (l & 63)) E[q][c] = xq;
      }
    }
    __syncthreads();
  }
  if (!solver) return;
  // The final plan and its cost.
  if (!solve(p.k)) return;
  double acc = 0.0;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const double bq = lane_f64(b8, q);
    const int j = min(jw + q, p.n - 1);               // E is zero past n
    double x = 0.0;
#pragma unroll
    for (int c = 0; c < kPersChunks; ++c) {
      const int i = c * 64 + lane;
      if (i < p.k) x = fma(sa[i] * E[q][c], double(p.C[size_t(j) * p.n + spick[i]]), x);
    }
    acc = fma(x, bq, acc);
  }
  acc = wave_sum(acc);
  if (lane == 0) smass[w] = acc;
  __syncthreads();
  if (tid == 0) {
    double x = 0.0;
    for (int q = 0; q < kWaves; ++q) x += smass[q];
    p.objpart[blk] = x;
  }
}

struct LitLayout {
  size_t E, a, b, r, colpart, scorepart, objpart, chosen, total;
  int kp, nrb, panels, strips;
};

LitLayout lit_layout(int64_t n, int64_t k) {
  LitLayout L;
  L.kp = int((k + 3) / 4 * 4);
  L.nrb = int((n + kLitRows - 1) / kLitRows);
  L.strips = int((n + kLitBlock - 1) / kLitBlock);
  L.panels = std::max(1, std::min(64, (512 + L.strips - 1) / L.strips));
  size_t o = 0;
  L.E = o;
  o = a256(o + size_t(n) * L.kp * 8);
  L.a = o;
  o = a256(o + size_t(L.kp) * 8);
  L.b = o;
  o = a256(o + size_t(n) * 8);
  L.r = o;
  o = a256(o + size_t(n) * 8);
  L.colpart = o;
  o = a256(o + size_t(L.nrb) * L.kp * 8);
  L.scorepart = o;
  o = a256(o + size_t(L.panels) * n * 8);
  L.objpart = o;
  o = a256(o + size_t(L.nrb) * 8);
  L.chosen = o;
  o = a256(o + size_t(n));
  L.total = o;
  return L;
}

// One solve over the first l retained tokens: `rounds` scaling rounds, the
// last one leaving b and the residual.
hipError_t solve(const LitDev& p, int l, int rounds, hipStream_t stream) {
  const int a_blocks = (l + kLitWaves - 1) / kLitWaves;
  lit_rows_kernel<<<p.nrb, kLitBlock, 0, stream>>>(p, l, 0);
  for (int it = 0; it < rounds; ++it) {
    lit_a_kernel<<<a_blocks, kLitBlock, 0, stream>>>(p, l);
    lit_rows_kernel<<<p.nrb, kLitBlock, 0, stream>>>(p, l, it + 1 < rounds ? 1 : 2);
  }
  return hipGetLastError();
}

// The persistent form's workspace: the words its blocks exchange, cleared
// before each launch, then the partial scores and objective parts.
constexpr size_t kPersWords = size_t(2) * kPersSolvers * kPersK + 2 * kPersN + 2 * kPersSolvers +
                              size_t(kPersBlocks) * kSlotStride + size_t(2) * kPersBlocks * kSlotStride;
bool lit_pers_serves(int64_t n, int64_t k) { return n <= kPersN && k <= kPersK; }
size_t lit_pers_bytes(int64_t n) {
  const size_t blocks = size_t((n + kPersScore - 1) / kPersScore);
  return a256(kPersWords * 8) + 256 + a256(size_t(kPersSolvers) * 8) + blocks * size_t(n) * 8;
}

// Runs the persistent form if the device can hold its grid and the stream is
// not being captured (the separate launches can be); *done says so.
hipError_t try_persistent(const LiteralParams& q, hipStream_t stream, bool* done) {
  *done = false;
  if (q.follow || q.rounds > kPersRounds || !lit_pers_serves(q.n, q.k) || q.workspace_bytes < lit_pers_bytes(q.n)) return hipSuccess;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &cap) != hipSuccess) {
    (void)hipGetLastError();
    return hipSuccess;
  }
  if (cap != hipStreamCaptureStatusNone) return hipSuccess;
  int dev = 0, cus = 0, per_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
  const void* kernel = reinterpret_cast<const void*>(lit_persistent_kernel);
  const size_t lds = size_t(kPersScore) * q.n * sizeof(float);
  if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kBlock, lds)) != hipSuccess) return e;
  const int blocks = (q.n + kPersScore - 1) / kPersScore;
  if (blocks > cus * per_cu) return hipSuccess;

  char* w = static_cast<char*>(q.workspace);
  LitPers p{};
  p.C = q.cost;
  p.v = q.capacity;
  p.n = q.n;
  p.k = q.k;
  p.rounds = q.rounds;
  p.eps = double(q.epsilon);
  p.u = 1.0 / double(q.k);
  p.selected = q.selected;
  p.step_score = q.step_score;
  p.step_residual = q.step_residual;
  p.col = reinterpret_cast<unsigned long long*>(w);
  p.r = p.col + size_t(2) * kPersSolvers * kPersK;
  p.mass = p.r + 2 * kPersN;
  p.flag = p.mass + 2 * kPersSolvers;
  p.cand = p.flag + size_t(kPersBlocks) * kSlotStride;
  w += a256(kPersWords * 8);
  p.abort = reinterpret_cast<unsigned int*>(w);
  w += 256;
  p.objpart = reinterpret_cast<double*>(w);
  w += a256(size_t(kPersSolvers) * 8);
  p.part = reinterpret_cast<double*>(w);
  const WaitPolicy wp = wait_policy();
  p.poll_limit = wp.limit;
  p.abort_init = wp.preset;
  p.solvers = (q.n + kPersRows - 1) / kPersRows;
  lit_pers_init_kernel<<<32, 256, 0, stream>>>(p, kPersWords);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  void* args[] = {&p};
  if ((e = hipLaunchCooperativeKernel(kernel, dim3(blocks), dim3(kBlock), args, lds, stream)) != hipSuccess) return e;
  if ((e = launch_mark_aborted(p.abort, p.selected, p.k, stream)) != hipSuccess) return e;
  if (q.objective) {
    LitDev d{};
    d.nrb = p.solvers;
    d.objpart = p.objpart;
    d.objective = q.objective;
    lit_objective_sum_kernel<<<1, 64, 0, stream>>>(d);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  *done = true;
  return hipSuccess;
}

}  // namespace

size_t sgs_literal_min_workspace_bytes(int64_t n, int64_t k) { return lit_layout(n, k).total; }

size_t sgs_literal_workspace_bytes(int64_t n, int64_t k) {
  return std::max(lit_layout(n, k).total, lit_pers_serves(n, k) ? lit_pers_bytes(n) : size_t(0));
}

hipError_t launch_sgs_literal(const LiteralParams& q, hipStream_t stream) {
  if (q.n < 1 || q.k < 1 || q.k > q.n || q.k > kLitMaxK || q.rounds < 1) return hipErrorInvalidValue;
  bool done = false;
  const hipError_t pe = try_persistent(q, stream, &done);
  if (pe != hipSuccess || done) return pe;
  const LitLayout L = lit_layout(q.n, q.k);
  char* w = static_cast<char*>(q.workspace);
  LitDev p;
  p.C = q.cost;
  p.v = q.capacity;
  p.n = q.n;
  p.k = q.k;
  p.kp = L.kp;
  p.eps = double(q.epsilon);
  p.u = 1.0 / double(q.k);
  p.E = reinterpret_cast<double*>(w + L.E);
  p.a = reinterpret_cast<double*>(w + L.a);
  p.b = reinterpret_cast<double*>(w + L.b);
  p.r = reinterpret_cast<double*>(w + L.r);
  p.colpart = reinterpret_cast<double*>(w + L.colpart);
  p.scorepart = reinterpret_cast<double*>(w + L.scorepart);
  p.objpart = reinterpret_cast<double*>(w + L.objpart);
  p.chosen = reinterpret_cast<unsigned char*>(w + L.chosen);
  p.selected = q.selected;
  p.follow = q.follow;
  p.step_score = q.step_score;
  p.step_residual = q.step_residual;
  p.objective = q.objective;
  p.nrb = L.nrb;
  p.panels = L.panels;
  p.strips = L.strips;

  hipError_t e;
  const int grid_n = std::min(1024, (q.n + 255) / 256);
  lit_init_kernel<<<grid_n, 256, 0, stream>>>(p);
  if (q.follow && !q.step_score && !q.step_residual) {
    // A trajectory to follow and no per-step output: only the final plan.
    lit_follow_kernel<<<(q.k + 255) / 256, 256, 0, stream>>>(p);
    for (int l = 1; l <= q.k; ++l) lit_append_kernel<<<grid_n, 256, 0, stream>>>(p, l);
  } else {
    for (int l = 0; l < q.k; ++l) {
      if (l > 0) {
        lit_append_kernel<<<grid_n, 256, 0, stream>>>(p, l);
        if ((e = solve(p, l, q.rounds, stream)) != hipSuccess) return e;
      }
      lit_score_kernel<<<dim3(L.strips, L.panels), kLitBlock, 0, stream>>>(p);
      lit_select_kernel<<<1, kSelectBlock, 0, stream>>>(p, l);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    lit_append_kernel<<<grid_n, 256, 0, stream>>>(p, q.k);
  }
  if ((e = solve(p, q.k, q.rounds, stream)) != hipSuccess) return e;
  if (q.objective) {
    lit_objective_kernel<<<L.nrb, kLitBlock, 0, stream>>>(p);
    lit_objective_sum_kernel<<<1, 64, 0, stream>>>(p);
  }
  return hipGetLastError();
}

}  // namespace cp
