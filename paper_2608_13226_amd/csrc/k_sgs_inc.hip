// Greedy coverage selection, incremental form (Sec. 3.5, Eq. 14-16).
//
// Same greedy as the dense sweep: step l picks
//   t_l = argmax_{c not chosen} gain(c),  gain(c) = sum_j v_j max(0, b_j - C_tm[j][c])
// and then b_j <- min(b_j, C_tm[j][t_l]).  Only the targets whose best cost
// drops at step l (the set J_l: C_tm[j][t_l] < b_j) change any gain, by
//   v_j (max(0, b'_j - C_tm[j][c]) - max(0, b_j - C_tm[j][c])),
// so the gains are computed once in full (b = c0) and then kept up to date
// from the rows of J_l alone: about sum_l |J_l| rows of C_tm are read instead
// of K full matrices.  Every term v_j max(0, b_j - C) is formed as in the
// dense sweep (the difference in float32, the product exactly in float64) and
// then rounded down onto a fixed-point grid of 2^-S, S chosen per launch so
// that c0 sum(v) stays below 2^62; gains are sums of these integers in 64
// bits.  Integer sums do not depend on their order, so the running gains are
// bit-identical to gains summed afresh from the current b (a gain that has
// dropped to zero is exactly zero), and equal gains go to the smaller index.
// The grid, about 2^-62 c0 sum(v), is finer than the rounding of a float64
// sum of the same terms.
//
// The fixed-point scale and the step-0 gains (b = c0) come from two ordinary
// kernels ahead of the greedy (inc_scale_kernel, inc_first_pass_kernel), which
// run with many more waves in flight than the greedy itself.  The greedy is
// one cooperative launch, one block of eight waves per compute unit.  Block b
// owns the rows and the columns [b W, (b + 1) W): the best costs b_j and
// capacities of its rows and the running gains of its columns stay in LDS for
// the whole launch.  Per step:
//   1. every block reads all blocks' candidates for the step (each block's
//      best unchosen column, published at the end of the previous step) and
//      takes the same winner;
//   2. it tests its own rows against the winner's column and writes the rows
//      that improve, compacted, to its slice of the change list (row, v,
//      old b, new b), then publishes the slice's length;
//   3. it reads every block's length, walks the whole change list (slices
//      in block order) and applies the changes to its columns' gains,
//      reading each changed row's segment over its columns (one coalesced
//      256-byte read per row and 64 columns); block 0 also applies them to the
//      objective, kept in the same fixed point;
//   4. it publishes the exact argmax of its unchosen columns.
//
// The exchanges and the fixed point are in sgs_exchange.h.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sgs_exchange.h"

namespace cp {
namespace {

constexpr int kBatch = 64;         // change-list entries a wave fetches per round
constexpr int kChunk = 16;         // of which the rows read together

// The greedy of one scene as run by block `blk` of the scene's `nb` blocks.
__device__ __forceinline__ void inc_body(const IncDev& a, int blk, int nb) {
  if (unfit(a)) return;
  extern __shared__ unsigned long long smem[];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lo = blk * a.W;
  const int cnt = max(0, min(a.n, lo + a.W) - lo);
  long long* sG = reinterpret_cast<long long*>(smem);             // [W] running gains
  float* sb = reinterpret_cast<float*>(sG + a.W);                  // [W] best costs of own rows
  float* sv = sb + a.W;                                            // [W] capacities of own rows
  unsigned char* ssel = reinterpret_cast<unsigned char*>(sv + a.W);       // [W] chosen columns
  __shared__ long long red[kBlock];
  __shared__ long long sg[kWaves];
  __shared__ int swt[kWaves];
  __shared__ unsigned long long su[kWaves];
  __shared__ int spre[kMaxBlocks + 1];        // slice offsets
  __shared__ int sflag;                       // abort seen while waiting for the winner
  __shared__ int slflag;                      // ... or for the slice lengths

  for (int i = tid; i < cnt; i += kBlock) {
    sb[i] = a.c0;
    sv[i] = a.v[lo + i];
    ssel[i] = 0;
  }

  // The fixed-point scale and the step-0 gains of the own columns (every row
  // at b = c0) come from the first-pass kernels: the gains as P partial sums
  // over row ranges, whose integer total does not depend on the split.
  const int S = *a.scale;
  for (int i = tid; i < cnt; i += kBlock) {
    long long g = 0;
    for (int q = 0; q < a.P; ++q) g += a.part[size_t(q) * a.n + lo + i];
    sG[i] = g;
  }
  __syncthreads();

  // Block 0 keeps the objective L = sum_j v_j b_j in the gains' fixed point,
  // starting from b = c0, as one running part per wave: a wave adds its share
  // of a step's changes without a barrier, and thread 0 totals the parts for
  // step l after the next step's first barrier (after the loop for the last).
  __shared__ long long sLw[kWaves];
  int obj_step = -1;
  if (blk == 0) {
    const long long x = fx_capacity_part(a.v, a.n, a.c0, S);
    const long long L0 = block_sum_i64(x, sg);
    if (tid < kWaves) sLw[tid] = tid == 0 ? L0 : 0;
  }

  publish_argmax(sG, ssel, lo, cnt, S, cand_slot(a.cand, 0, blk), epoch_of(0), su);

  for (int step = 0; step < a.k; ++step) {
    // Some block has a candidate while unchosen columns remain; the clamp
    // only keeps a broken slot from addressing past the matrix.
    const int tw = read_winner(cand_slot(a.cand, step & 1, 0), epoch_of(step), nb, a.abort, a.poll_limit, su, &sflag);
    if (tw < 0) break;
    if (blk == 0 && tid == 0 && obj_step >= 0 && a.step_obj) {
      long long L = 0;
#pragma unroll
      for (int q = 0; q < kWaves; ++q) L += sLw[q];
      a.step_obj[obj_step] = fx_to_double(L, S);
    }
    const int t = min(tw, a.n - 1);
    if (t >= lo && t < lo + cnt && tid == 0) {
      ssel[t - lo] = 1;
      a.selected[step] = t;
      if (a.step_gain) a.step_gain[step] = fx_to_double(sG[t - lo], S);
    }

    // 1. Own rows that the pick improves, compacted into the block's slice.
    int base = 0;
    unsigned long long* mine = a.list + size_t(blk) * a.W * 2;
    for (int i0 = 0; i0 < cnt; i0 += kBlock) {
      const int i = i0 + tid;
      float cv = 0.f, bo = 0.f;
      bool hit = false;
      if (i < cnt) {
        cv = a.C[size_t(lo + i) * a.n + t];
        bo = sb[i];
        hit = cv < bo;
      }
      const unsigned long long m = __ballot(hit);
      const int rank = __popcll(m & ((1ull << lane) - 1ull));
      if (lane == 0) swt[w] = __popcll(m);
      __syncthreads();
      int off = base, tot = 0;
#pragma unroll
      for (int q = 0; q < kWaves; ++q) {
        if (q < w) off += swt[q];
        tot += swt[q];
      }
      if (hit) {
        const int slot = off + rank;
        put(mine + size_t(slot) * 2,
            (unsigned long long)(unsigned int)(lo + i) | ((unsigned long long)__float_as_uint(sv[i]) << 32));
        put(mine + size_t(slot) * 2 + 1,
            (unsigned long long)__float_as_uint(bo) | ((unsigned long long)__float_as_uint(cv) << 32));
        sb[i] = cv;
        if (a.assign) a.assign[lo + i] = t;
      }
      base += tot;
      __syncthreads();
    }
    // The barrier above completed this block's list writes.
    if (tid == 0) put(lens_slot(a.lens, blk), ((unsigned long long)(step + 1) << 32) | unsigned(base));

    // The last step's changes only feed the objective, kept by block 0.
    if (step + 1 == a.k && blk != 0) break;

    // 2. Every block's slice length (thread i waits for block i), and the
    // slices' offsets in the flattened change list.
    {
      if (tid == 0) slflag = 0;
      __syncthreads();
      int c = 0;
      if (tid < nb) {
        unsigned long long x;
        const unsigned int round = unsigned(step + 1);
        if (wait_slot(lens_slot(a.lens, tid), a.abort, a.poll_limit,
                      [round](unsigned long long v) { return (v >> 32) == round; }, x))
          c = int(x & 0xffffffffull);
        else
          slflag = 1;
      }
      const int incl = block_inclusive_scan(c, swt);
      if (tid < nb) spre[tid + 1] = incl;
      if (tid == 0) spre[0] = 0;
      __syncthreads();
    }
    if (slflag) break;
    const int total = spre[nb];

    // 3. Apply the changes to the own columns' gains.  Each lane of a round
    // locates and fetches one entry; the entries are then broadcast and every
    // lane reads its column of each entry's row.
    long long dobj = 0;
    for (int cc = 0; cc < cnt; cc += 64) {
      const bool colok = cc + lane < cnt;
      const int col = lo + cc + lane;
      long long g = 0;
      // Rounds of up to kBatch entries per wave, the list split evenly over
      // the waves.
      const int per = min(kBatch, (total + kWaves - 1) / kWaves);
      for (int e0 = w * per; e0 < total; e0 += kWaves * per) {
        const int e = e0 + lane;
        unsigned long long h0 = 0ull, h1 = 0ull;
        if (lane < per && e < total) {
          int s0 = 0, s1 = nb;   // spre[s0] <= e < spre[s1]
          while (s1 - s0 > 1) {
            const int mid = (s0 + s1) >> 1;
            if (spre[mid] <= e) s0 = mid;
            else s1 = mid;
          }
          const unsigned long long* src = a.list + (size_t(s0) * a.W + size_t(e - spre[s0])) * 2;
          h0 = get(src);
          h1 = get(src + 1);
        }
        const int m = min(per, total - e0);
        // Entry u is broadcast from lane u with readlane (u is uniform), in
        // chunks of kChunk whose row reads are in flight together.
        const int hj = int(h0 & 0xffffffffull);
        const int hbo = int(h1 & 0xffffffffull), hbn = int(h1 >> 32);
        // Each lane's entry capacity scaled once for fx_scaled.
        const long long hvs = __double_as_longlong(fx_scale(double(__uint_as_float(unsigned(h0 >> 32))), S));
        for (int u0 = 0; u0 < m; u0 += kChunk) {
          float x[kChunk];
#pragma unroll
          for (int i = 0; i < kChunk; ++i) {
            x[i] = 0.f;
            if (u0 + i < m && colok) {
              const int j = __builtin_amdgcn_readlane(hj, u0 + i);
              x[i] = a.C[size_t(j) * a.n + col];
            }
          }
#pragma unroll
          for (int i = 0; i < kChunk; ++i) {
            if (u0 + i < m) {
              // A column that cost at least the old best contributes 0 before
              // and after (new best < old best).
              const float bo = __int_as_float(__builtin_amdgcn_readlane(hbo, u0 + i));
              if (x[i] < bo) {
                const float bn = __int_as_float(__builtin_amdgcn_readlane(hbn, u0 + i));
                const double vs = __longlong_as_double(
                    (long long)(((unsigned long long)(unsigned)__builtin_amdgcn_readlane(int(hvs >> 32), u0 + i) << 32) |
                                (unsigned)__builtin_amdgcn_readlane(int(hvs), u0 + i)));
                g += (long long)(fx_scaled(vs, fmaxf(bn - x[i], 0.f)) - fx_scaled(vs, bo - x[i]));
              }
            }
          }
        }
        if (blk == 0 && cc == 0 && lane < per && e < total) {
          const double vj = double(__uint_as_float(unsigned(h0 >> 32)));
          const float bo = __uint_as_float(unsigned(h1 & 0xffffffffull));
          const float bn = __uint_as_float(unsigned(h1 >> 32));
          dobj += fx(vj * double(bn), S) - fx(vj * double(bo), S);
        }
      }
      red[tid] = g;
      __syncthreads();
      if (tid < 64 && cc + tid < cnt) {
        long long s = sG[cc + tid];
#pragma unroll
        for (int q = 0; q < kWaves; ++q) s += red[q * 64 + tid];
        sG[cc + tid] = s;
      }
      __syncthreads();
    }
    if (blk == 0) {
      dobj = wave_sum_i64(dobj);
      if (lane == 0) sLw[w] += dobj;
      obj_step = step;
    }

    // 4. This block's candidate for the next step.
    if (step + 1 < a.k)
      publish_argmax(sG, ssel, lo, cnt, S, cand_slot(a.cand, (step + 1) & 1, blk),
                     epoch_of(step + 1), su);
  }
  __syncthreads();
  if (blk == 0 && tid == 0 && obj_step >= 0 && a.step_obj) {
    long long L = 0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) L += sLw[q];
    a.step_obj[obj_step] = fx_to_double(L, S);
  }
}

// ---------------------------------------------------------------------------
// Rows form of the same greedy, for scenes whose n best costs fit in LDS.
//
// The exchange form learns J_l from the owners of the rows (a pass over the
// own rows, an exchange of slice lengths, a walk of the change list).  Here
// every block keeps all n best costs b_j in LDS and finds J_l itself: it
// reads the winner's costs to every target, C(t_l, j) for all j, as one
// contiguous row of a source-major copy T of the cost (T[s][j] = C(s, j)),
// tests each against b_j, and applies the rows that improve straight away.
// Every block then holds the identical J_l and the identical b, a step needs
// one exchange (the candidates) instead of two, and no block reads another's
// list.  T is written by the first-pass kernel, which reads the whole cost in
// column strips for the step-0 gains anyway.
//
// Per step and wave: the wave's chunks of the winner's row (256 targets a
// load, 16 bytes a lane) are loaded together; a chunk without a hit costs one
// LDS read and four compares; hits are compacted into the wave's list in LDS
// (target, old b, new b) and their rows' segments over the block's columns
// are read 16 rows at a time.  The block's columns' deltas are then summed
// over the waves in wave order, as in the exchange form, and are the same
// integers, so both forms take the same picks.
constexpr int kRowsMaxN = 32768;   // 128 KB of best costs in LDS
constexpr int kRowsMaxW = 128;     // columns per block: two per lane
constexpr int kRowChunk = 256;     // targets per wave-load of the winner's row
constexpr int kList = 128;         // hits a wave collects before applying them (dense steps)
constexpr int kCap = kList * kWaves;   // hits a block lists in one step

int rows_ldt(int64_t n) { return int((n + kRowChunk - 1) / kRowChunk * kRowChunk); }

// Fixed-point scale, the same in every block (same sum, same order): every
// partial gain is at most c0 sum(v) < 2^(62 - S), and every single term
// v_j d 2^S (0 <= d <= c0) at most c0 max(v) 2^S < 2^52, which fx_diff
// needs.
__device__ __forceinline__ int fixed_scale(const IncDev& a, double* sd) {
  double x = 0.0, m = 0.0;
  // Thread t adds v[t], v[t + kBlock], ... in that order; the loads of
  // eight of them go out together (indices past n read v[n - 1], unused).
  constexpr int U = 8;
  for (int j0 = threadIdx.x; j0 < a.n; j0 += kBlock * U) {
    float vv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) vv[u] = a.v[min(j0 + u * kBlock, a.n - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j0 + u * kBlock < a.n) {
        x += double(vv[u]);
        m = fmax(m, double(vv[u]));
      }
  }
  const double M = double(a.c0) * block_sum_all(x, sd);
  const double Mt = double(a.c0) * block_max_all(m, sd);
  int S = 0;
  if (M > 0.0) {
    int e = 0;
    (void)__builtin_frexp(M, &e);   // M < 2^e
    S = 62 - e;
    (void)__builtin_frexp(Mt, &e);  // 0 < Mt <= M
    S = min(S, 52 - e);
  }
  return S;
}

// Predicting the next winner (rows schedule, at most 64 columns a block).
// Each block publishes two words in its slot: its best key (word 0) and its
// second-best key (word 1), each with the exchange's epoch bit.  After a
// step's exchange every block knows, for the runner-up r (the best candidate
// outside the winner's block), a lower bound on its fixed-point gain (from
// its key), and an upper bound U on every other candidate's truncated gain:
// the best keys of all blocks but the winner's and r's, and the second-best
// keys of those two (a block's other columns are at most its second best, and
// gains only fall).  While applying the step's hits every block also sums
// r's changes from the same terms, so every block holds the same lower bound
// on r's gain after the step; if its truncated gain is strictly above U, r is
// the next winner (whatever the indices), every block knows it, and the next
// step runs without an exchange, on r's row of T loaded during this step.
// A lower bound on the fixed-point gain g behind a key: the key keeps the
// top bits of the float64 value of g 2^-S (rounded to nearest from 64 bits,
// then truncated), so scaling it back can exceed g by at most half a unit in
// the 53rd bit, which the bound takes off.
__device__ __forceinline__ long long key_gain_floor(unsigned long long key, int S) {
  const double d = __longlong_as_double((long long)((key >> kIndexBits) << (kIndexBits + 1)));
  const long long G = (long long)__builtin_ldexp(d, S);
  return max(0ll, G - (G >> 52) - 1);
}

// The best costs that the rows kernel hands to the list phase, ldt floats
// beside the lists' lengths: both lie in the compact form's change lists
// (16 (n + kMaxBlocks) bytes), which the rows form does not use.
__host__ __device__ __forceinline__ size_t llen_words(int n) { return (size_t(n) + 63) / 64 * 64; }
__device__ __forceinline__ float* list_ho_b(const IncDev& a) { return reinterpret_cast<float*>(a.llen + llen_words(a.n)); }

constexpr int kTrackMax = 256;   // hits of a step that still tracks the runner-up

// The step-0 gains of a block's columns [lo, lo + cnt) from the P partial
// sums part[q][column] (64-bit integers, so the split does not matter):
// thread (column tid % 64, group tid / 64) adds partials group, group +
// kWaves, ..., eight loads in flight, then the groups' sums are added in
// LDS.  P is 3 after the first pass, n / 64 after the fused epilogue.
__device__ __forceinline__ void init_gains(const IncDev& a, long long* sG, int lo, int cnt, long long* red) {
  const int tid = threadIdx.x, g = tid >> 6;
  for (int i0 = 0; i0 < cnt; i0 += 64) {
    const int i = i0 + (tid & 63);
    const int col = lo + min(i, cnt - 1);
    long long x = 0;
    for (int q0 = g; q0 < a.P; q0 += 8 * kWaves) {
      long long v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = a.part[size_t(min(q0 + u * kWaves, a.P - 1)) * a.n + col];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (q0 + u * kWaves < a.P) x += v[u];
    }
    red[tid] = x;
    __syncthreads();
    if (tid < 64 && i0 + tid < cnt) {
      long long t = 0;
#pragma unroll
      for (int r = 0; r < kWaves; ++r) t += red[r * 64 + tid];
      sG[i0 + tid] = t;
    }
    __syncthreads();
  }
}

// NG 64-column groups per block (W <= 64 NG); RL chunk loads per wave and
// step (n <= kRowChunk kWaves RL).
template <int NG, int RL>
__device__ __forceinline__ void rows_body(const IncDev& a, int blk, int nb) {
  extern __shared__ unsigned long long smem[];
  // Hits a block lists in one step: with one column group the list is four
  // times kCap (48 KB of LDS beside the 64 KB of best costs), which puts all
  // but the first dense steps in one round; two groups keep 128 KB of best
  // costs and the short list.
  constexpr int kCapR = (NG == 1 ? 4 : 1) * kCap;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lo = blk * a.W;
  const int cnt = max(0, min(a.n, lo + a.W) - lo);
  long long* sG = reinterpret_cast<long long*>(smem);             // [W] running gains (W rounded up to even)
  float* sball = reinterpret_cast<float*>(sG + ((a.W + 1) & ~1));  // [ldt] b_j, 16-byte aligned; -inf past n
  unsigned char* ssel = reinterpret_cast<unsigned char*>(sball + a.ldt);   // [W] chosen columns
  __shared__ long long red[kBlock];
  __shared__ long long sg[kWaves];
  __shared__ unsigned long long su[kWaves];
  __shared__ int sflag[2];
  __shared__ int lj[kCapR];                    // hit list: target
  __shared__ float lbo[kCapR];                 // old best cost
  __shared__ float lbn[kCapR];                 // new best cost
  __shared__ int scnt[2];                     // hits listed in steps of each parity
  __shared__ int schunk[kRowsMaxN / kRowChunk];   // dense steps: hits per chunk, then their offsets
  if (tid == 0) scnt[0] = scnt[1] = 0;
  // Prediction of the next winner (one column group only): every block's
  // slot words of the last exchange and the waves' parts of the runner-up's
  // change in the step.
  constexpr bool kSpec = NG == 1;
  __shared__ unsigned long long sk1[kSpec ? kMaxBlocks : 1], sk2[kSpec ? kMaxBlocks : 1], sk3[kSpec ? kMaxBlocks : 1];
  __shared__ long long sdr[kWaves];

  if (unfit(a)) return;
  // After the early kernel the first step is the one it stopped before.
  if (a.start && *a.abort) return;
  const int k_begin = a.start ? int(*a.start) : a.k_begin;
  const bool resume = k_begin > 0;
  if (resume && *a.abort) return;             // the launch before it gave up
  // The fixed-point scale, the step-0 gains (as P partial sums over row
  // ranges) and T come from the first-pass kernels.
  const int S = *a.scale;
  if (resume) {
    for (int j = tid; j < a.ldt; j += kBlock) sball[j] = a.ho_b[j];
    for (int i = tid; i < cnt; i += kBlock) {
      ssel[i] = a.ho_sel[lo + i];
      sG[i] = a.ho_gain[lo + i];
    }
  } else {
    for (int j = tid; j < a.ldt; j += kBlock) sball[j] = j < a.n ? a.c0 : -__builtin_inff();
    for (int i = tid; i < cnt; i += kBlock) ssel[i] = 0;
    init_gains(a, sG, lo, cnt, red);
  }
  __syncthreads();

  // Block 0 keeps the objective as one running part per wave (as in the
  // exchange form).
  __shared__ long long sLw[kWaves];
  int obj_step = k_begin - 1;
  if (blk == 0) {
    long long L0 = 0;
    if (resume) {
      L0 = a.ho_misc[0];
    } else {
      const long long x = fx_capacity_part(a.v, a.n, a.c0, S);
      L0 = block_sum_i64(x, sg);
    }
    if (tid < kWaves) sLw[tid] = tid == 0 ? L0 : 0;
  }

  // Slot sets and epochs count exchanges, which predicted steps skip.  After
  // the early kernel the first exchange's candidates are published.
  int xc = resume ? int(a.ho_misc[1]) : 0;
  if (!resume) {
    if (kSpec)
      publish_rows<true>(a, sG, ssel, lo, cnt, S, cand_slot(a.cand, 0, blk), epoch_of(0));
    else
      publish_argmax(sG, ssel, lo, cnt, S, cand_slot(a.cand, 0, blk), epoch_of(0), su);
  }

  const int nch = a.ldt / kRowChunk;
  bool predicted = false;     // this step's winner was predicted (no exchange)
  int tpred = -1;
  f32x4 xr2[RL];              // the predicted winner's row, loaded during the previous step
  // The runner-up of the last exchange, the same in every wave and block
  // (-1 when the step has none: it was predicted itself, or had many hits),
  // the lower bound on its gain with the changes since, and the truncated
  // gain it must exceed.
  int rn = -1;
  long long racc = 0;
  unsigned long long rub = 0ull;
  for (int step = k_begin; step < a.k_end; ++step) {
    int tw;
    if (predicted) {
      __syncthreads();
      tw = tpred;
    } else {
      tw = kSpec ? read_winner_rows<true>(a, cand_slot(a.cand, xc & 1, 0), epoch_of(xc), nb, su, sflag, sk1, sk2, sk3)
                 : read_winner(cand_slot(a.cand, xc & 1, 0), epoch_of(xc), nb, a.abort, a.poll_limit, su, sflag);
      ++xc;
    }
    if (tw < 0) break;
    if (blk == 0 && tid == 0 && obj_step >= 0 && a.step_obj) {
      long long L = 0;
#pragma unroll
      for (int q = 0; q < kWaves; ++q) L += sLw[q];
      a.step_obj[obj_step] = fx_to_double(L, S);
    }
    const int t = min(tw, a.n - 1);
    if (t >= lo && t < lo + cnt && tid == 0) {
      ssel[t - lo] = 1;
      a.selected[step] = t;
      if (a.step_gain) a.step_gain[step] = fx_to_double(sG[t - lo], S);
    }

    // The wave's chunks of the winner's row, all loads in flight together
    // (already loaded when the winner was predicted).
    const f32x4* row = reinterpret_cast<const f32x4*>(a.T + size_t(t) * a.ldt);
    f32x4 xr[RL];
#pragma unroll
    for (int i = 0; i < RL; ++i)
      if (w + i * kWaves < nch) xr[i] = predicted ? xr2[i] : row[(w + i * kWaves) * (kRowChunk / 4) + lane];

    // After an exchange every wave finds the runner-up while the row is in
    // flight.  Blocks own W consecutive columns, so the winner's is t / W.
    if (kSpec) {
      rn = -1;
      if (!predicted) {
        const int bt = block_of(a, t);
        unsigned long long k[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int b = lane + 64 * q;
          k[q] = (b < nb && b != bt) ? sk1[b] : 0ull;
        }
        const unsigned long long kr = wave_max_u64(max(max(k[0], k[1]), max(k[2], k[3])));
        if (kr > kNoCandidate) {
          rn = min(int(kIndexMask - (kr & kIndexMask)), a.n - 1);
          racc = key_gain_floor(kr, S);
          const int br = block_of(a, rn);
#pragma unroll
          for (int q = 0; q < 4; ++q) k[q] = (lane + 64 * q) == br ? 0ull : k[q];
          const unsigned long long u = wave_max_u64(max(max(k[0], k[1]), max(k[2], k[3])));
          rub = max(u, max(sk2[bt], sk2[br])) >> kIndexBits;
        }
      }
    }

    long long g[NG];
#pragma unroll
    for (int q = 0; q < NG; ++q) g[q] = 0;
    long long dobj = 0;
    long long dr = 0;           // this wave's part of the runner-up's change
    // Applies listed hits base .. base + m to the wave's partial gains (and,
    // in block 0, to the objective), and records them in assign and (with
    // setb) in b.
    auto apply = [&](int base, int m, bool setb) {
      // Lane u < kChunk of a batch holds entry e0 + u and its capacity; the
      // entries are broadcast with readlane.  The next batch's entries and
      // row reads are issued before the current batch's terms are summed.
      int jl = 0;
      float bol = 0.f, bnl = 0.f, vl = 0.f;
      float rl = 0.f;
      float xc[kChunk][NG];
      auto fetch = [&](int e0) {
        const int nbt = min(kChunk, base + m - e0);
        jl = 0;
        bol = bnl = vl = 0.f;
        rl = 0.f;
        if (lane < nbt) {
          jl = lj[e0 + lane];
          bol = lbo[e0 + lane];
          bnl = lbn[e0 + lane];
          vl = a.v[jl];
          if (kSpec && rn >= 0) rl = a.C[size_t(jl) * a.n + rn];   // C(r, j): the runner-up's cost to the entry
        }
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
          const int j = __builtin_amdgcn_readlane(jl, u);
#pragma unroll
          for (int q = 0; q < NG; ++q)
            xc[u][q] = (u < nbt && q * 64 + lane < cnt) ? a.C[size_t(j) * a.n + lo + q * 64 + lane] : 0.f;
        }
      };
      if (m > 0) fetch(base);
      for (int e0 = base; e0 < base + m; e0 += kChunk) {
        const int nbt = min(kChunk, base + m - e0);
        const int cj = jl;
        const float cbo = bol, cbn = bnl;
        // Each lane's entry capacity scaled once for fx_diff (0 past the
        // batch, where v was not read).
        const double cvs = fx_scale(double(vl), S);
        const long long cvb = __double_as_longlong(cvs);
        const float cr = rl;
        float cx[kChunk][NG];
#pragma unroll
        for (int u = 0; u < kChunk; ++u)
#pragma unroll
          for (int q = 0; q < NG; ++q) cx[u][q] = xc[u][q];
        if (e0 + kChunk < base + m) fetch(e0 + kChunk);
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
          if (u < nbt) {
            const float bo = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cbo), u));
            const float bn = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cbn), u));
            const double vs = __longlong_as_double(
                (long long)(((unsigned long long)(unsigned)__builtin_amdgcn_readlane(int(cvb >> 32), u) << 32) |
                            (unsigned)__builtin_amdgcn_readlane(int(cvb), u)));
#pragma unroll
            for (int q = 0; q < NG; ++q) {
              // A column that cost at least the old best contributes 0
              // before and after.
              const float xx = cx[u][q];
              if (q * 64 + lane < cnt && xx < bo) g[q] += fx_diff(vs, fmaxf(bn - xx, 0.f), bo - xx);
            }
          }
        }
        // The batch's targets, one lane each: objective (block 0), the
        // runner-up's change, b and assign.
        if (lane < nbt) {
          if (kSpec && rn >= 0 && cr < cbo) dr += fx_diff(cvs, fmaxf(cbn - cr, 0.f), cbo - cr);
          if (blk == 0) dobj += fx_diff(cvs, cbn, cbo);
          if (setb) sball[cj] = cbn;
          if (a.assign && unsigned(cj - lo) < unsigned(cnt)) a.assign[cj] = t;
        }
      }
    };

    // Fast path: the waves list the hits of their chunks in one block-wide
    // list (a chunk's hits reserve their places with one LDS atomic), and
    // after a barrier each wave applies an equal share of it: the targets a
    // pick improves lie close together, in few chunks of few waves.
    const int par = step & 1;
#pragma unroll
    for (int i = 0; i < RL; ++i) {
      const int q0 = w + i * kWaves;
      if (q0 < nch) {
        const int j0 = q0 * kRowChunk + 4 * lane;     // this lane's four targets
        const f32x4 bo = *reinterpret_cast<const f32x4*>(sball + j0);
        const f32x4 x = xr[i];
        const unsigned long long m0 = __ballot(x[0] < bo[0]), m1 = __ballot(x[1] < bo[1]);
        const unsigned long long m2 = __ballot(x[2] < bo[2]), m3 = __ballot(x[3] < bo[3]);
        if ((m0 | m1 | m2 | m3) != 0ull) {
          const unsigned long long lt = (1ull << lane) - 1ull;
          const int tot = __popcll(m0) + __popcll(m1) + __popcll(m2) + __popcll(m3);
          int at = 0;
          if (lane == 0) at = atomicAdd(&scnt[par], tot);
          at = __builtin_amdgcn_readlane(at, 0);
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const unsigned long long mk = c == 0 ? m0 : c == 1 ? m1 : c == 2 ? m2 : m3;
            const int e = at + __popcll(mk & lt);
            if (((mk >> lane) & 1ull) && e < kCapR) {
              lj[e] = j0 + c;
              lbo[e] = bo[c];
              lbn[e] = x[c];
            }
            at += __popcll(mk);
          }
        }
      }
    }
    __syncthreads();
    const int total = scnt[par];
    // Early steps improve many targets; tracking the runner-up there costs
    // more than it saves.
    if (total > kTrackMax) rn = -1;
    if (tid == 0) scnt[par ^ 1] = 0;   // last read in the previous step, next used in the next
    if (total <= kCapR) {
      const int per = (total + kWaves - 1) / kWaves;
      const int e0 = min(total, w * per);
      apply(e0, min(total, e0 + per) - e0, true);
    } else {
      // Dense step (early in the greedy): the list is built and applied in
      // rounds of kCapR entries, each entry's place fixed by the hit counts
      // of the chunks before it, and every round is shared evenly by the
      // waves.  b keeps its old values until the last round (the hit test is
      // repeated each round), then takes the new ones.
      for (int q0 = w; q0 < nch; q0 += kWaves) {
        const int j0 = q0 * kRowChunk + 4 * lane;
        const f32x4 bo = *reinterpret_cast<const f32x4*>(sball + j0);
        const f32x4 x = row[q0 * (kRowChunk / 4) + lane];
        const int c = __popcll(__ballot(x[0] < bo[0])) + __popcll(__ballot(x[1] < bo[1])) +
                      __popcll(__ballot(x[2] < bo[2])) + __popcll(__ballot(x[3] < bo[3]));
        if (lane == 0) schunk[q0] = c;
      }
      __syncthreads();
      if (w == 0) {
        // Exclusive prefix of the chunk counts, two chunks a lane.
        const int c0 = 2 * lane < nch ? schunk[2 * lane] : 0;
        const int c1 = 2 * lane + 1 < nch ? schunk[2 * lane + 1] : 0;
        const int incl = wave_scan_incl(c0 + c1);
        if (2 * lane < nch) schunk[2 * lane] = incl - c0 - c1;
        if (2 * lane + 1 < nch) schunk[2 * lane + 1] = incl - c1;
      }
      __syncthreads();
      for (int r0 = 0; r0 < total; r0 += kCapR) {
        for (int q0 = w; q0 < nch; q0 += kWaves) {
          const int j0 = q0 * kRowChunk + 4 * lane;
          const f32x4 bo = *reinterpret_cast<const f32x4*>(sball + j0);
          const f32x4 x = row[q0 * (kRowChunk / 4) + lane];
          int at = schunk[q0] - r0;
          for (int c = 0; c < 4; ++c) {
            const bool hit = x[c] < bo[c];
            const unsigned long long mk = __ballot(hit);
            const int e = at + __popcll(mk & ((1ull << lane) - 1ull));
            if (hit && e >= 0 && e < kCapR) {
              lj[e] = j0 + c;
              lbo[e] = bo[c];
              lbn[e] = x[c];
            }
            at += __popcll(mk);
          }
        }
        __syncthreads();
        const int m = min(kCapR, total - r0);
        const int per = (m + kWaves - 1) / kWaves;
        const int e0 = min(m, w * per);
        apply(e0, min(m, e0 + per) - e0, false);
        __syncthreads();
      }
      for (int q0 = w; q0 < nch; q0 += kWaves) {
        const int j0 = q0 * kRowChunk + 4 * lane;
        f32x4 b = *reinterpret_cast<const f32x4*>(sball + j0);
        const f32x4 x = row[q0 * (kRowChunk / 4) + lane];
#pragma unroll
        for (int c = 0; c < 4; ++c) b[c] = x[c] < b[c] ? x[c] : b[c];
        *reinterpret_cast<f32x4*>(sball + j0) = b;
      }
    }

    // The runner-up's row for the next step if it is confirmed: issued after
    // the step's own loads so that none of their waits includes it.
    if (kSpec && rn >= 0) {
      const long long d = wave_sum_i64(dr);
      if (lane == 0) sdr[w] = d;
      const f32x4* rowr = reinterpret_cast<const f32x4*>(a.T + size_t(rn) * a.ldt);
#pragma unroll
      for (int i = 0; i < RL; ++i)
        if (w + i * kWaves < nch) xr2[i] = rowr[(w + i * kWaves) * (kRowChunk / 4) + lane];
    }
    // The waves' partial gains, added in wave order by wave 0.  With one
    // column group wave 0 then publishes the candidate on its own (the next
    // step begins with a barrier); with two the general publish reads every
    // column after a barrier.
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      red[tid] = g[q];
      __syncthreads();
      if (tid < 64 && q * 64 + tid < cnt) {
        const int c = q * 64 + tid;
        long long s = sG[c];
#pragma unroll
        for (int r = 0; r < kWaves; ++r) s += red[r * 64 + tid];
        sG[c] = s;
      }
      if (NG > 1) __syncthreads();
    }
    if (blk == 0) {
      dobj = wave_sum_i64(dobj);
      if (lane == 0) sLw[w] += dobj;
      obj_step = step;
    }

    // The lower bound on the runner-up's gain after the step, the same in
    // every block: above the bound on all others, it is the next winner.
    bool next = false;
    if (kSpec && rn >= 0) {
#pragma unroll
      for (int q = 0; q < kWaves; ++q) racc += sdr[q];
      next = step + 1 < a.k_end && racc > 0 && (pack_key(fx_to_double(racc, S), rn) >> kIndexBits) > rub;
    }
    if (step + 1 < a.k_end && !next) {
      if (kSpec)
        publish_rows<true>(a, sG, ssel, lo, cnt, S, cand_slot(a.cand, xc & 1, blk), epoch_of(xc));
      else
        publish_argmax(sG, ssel, lo, cnt, S, cand_slot(a.cand, xc & 1, blk), epoch_of(xc), su);
    }
    predicted = next;
    tpred = rn;
  }
  __syncthreads();
  if (blk == 0 && tid == 0 && obj_step >= 0 && a.step_obj) {
    long long L = 0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) L += sLw[q];
    a.step_obj[obj_step] = fx_to_double(L, S);
  }
  // Hand the state over to the list phase, which starts with an exchange of
  // its own.  The best costs go to a place of their own: a launch that resumed
  // with one step left, or two of which the second was predicted, waits for no
  // exchange after its first, whose candidates the early kernel published, so
  // block 0 can be here before a late block has read ho_b.
  if (a.k_end < a.k) {
    for (int i = tid; i < cnt; i += kBlock) {
      a.ho_gain[lo + i] = sG[i];
      a.ho_sel[lo + i] = ssel[i];
    }
    if (blk == 0) {
      float* bo = list_ho_b(a);
      for (int j = tid; j < a.ldt; j += kBlock) bo[j] = sball[j];
      if (tid == 0) {
        long long L = 0;
#pragma unroll
        for (int q = 0; q < kWaves; ++q) L += sLw[q];
        a.ho_misc[0] = L;
      }
    }
  }
}

__global__ __launch_bounds__(kBlock) void sgs_inc_kernel(IncDev a) { inc_body(a, blockIdx.x, gridDim.x); }

template <int NG, int RL>
__global__ __launch_bounds__(kBlock) void sgs_rows_kernel(IncDev a) { rows_body<NG, RL>(a, blockIdx.x, gridDim.x); }

// ---------------------------------------------------------------------------
// The rows schedule's early steps.
//
// A pick early in the greedy lowers the best cost of thousands of targets
// (about a fifth of all targets in each of the first 16 steps at N = 16384),
// and the rows kernel has every block read its own 64 columns of each such
// target's row of the cost: a 256-byte piece of thousands of rows per block
// and step, which the memory system serves at well under half its streaming
// rate.  Here the step's hits are split instead.  Every block still finds all
// of them from the winner's row of T (each block keeps every best cost);
// block b then takes the b-th equal share of the hit list (in target order),
// reads its targets' whole rows of the cost (contiguous, 64 KB each at
// N = 16384) and sums the gain changes of all n columns, the same 64-bit
// fixed-point terms as the rows kernel, into registers.  It writes the sums
// to its row of a [blocks] x [n] table, with the objective's change of its
// share after them, and raises its flag for the step; every block then adds,
// for its own columns, the rows of all blocks whose share was not empty.  The
// gains are the same integers as in the rows kernel (integer sums do not
// depend on their order), so the picks are the same.
//
// The kernel runs while a step improves at least kEarlyMinHits targets, and
// at most until the lists take over (or to the end), then hands its state
// to the rows kernel as the rows kernel hands it to the list kernel, with the
// next step in ho_misc[2].  A thread holds the changes of n / kBlock columns
// (n <= kEarlyMaxN).
constexpr int kEarlyMaxN = kRowChunk * kWaves * 8;    // 16384, the one-group rows kernel's reach
constexpr int kEarlyCols = kEarlyMaxN / kBlock;       // columns per thread: 32
constexpr int kEarlyPass = 8;                         // of which one pass over the share sums
constexpr int kEarlyDepth = 4;                        // rows whose loads are in flight
constexpr int kEarlyShare = 128;                      // hits a block takes per step at most
constexpr int kEarlyMinHits = 512;                    // steps with fewer hits go back to the rows kernel

int early_ldp(int64_t n) { return int((n + 1 + 63) / 64 * 64); }
// Up to kEarlyMinN tokens the rows kernel serves the first steps as well, in
// one launch less (the prune of 1024 tokens, K = 102: 0.54 ms with the early
// kernel's steps of 24 us, 0.39 without; 2048 tokens, K = 409: 0.97 and 0.94).
constexpr int kEarlyMinN = 2048;
bool early_for(int64_t n, int W) { return n > kEarlyMinN && n <= kEarlyMaxN && W <= kRowsMaxW; }

// NG 64-column groups per block, as in the rows kernel that continues.
template <int NG>
__device__ __forceinline__ void early_body(const IncDev& a, int blk, int nb) {
  if (!a.epart) return;                               // a scene of a batch without early steps
  extern __shared__ unsigned long long smem[];
  constexpr int RL = 8;                               // chunk loads per wave: n <= kRowChunk kWaves RL
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lo = blk * a.W;
  const int cnt = max(0, min(a.n, lo + a.W) - lo);
  long long* sG = reinterpret_cast<long long*>(smem);             // [W] running gains (W rounded up to even)
  float* sball = reinterpret_cast<float*>(sG + ((a.W + 1) & ~1));  // [ldt] b_j; -inf past n
  unsigned char* ssel = reinterpret_cast<unsigned char*>(sball + a.ldt);   // [W] chosen columns
  __shared__ long long red[NG * kBlock];
  __shared__ unsigned long long su[kWaves];
  __shared__ unsigned long long sk1[NG == 1 ? kMaxBlocks : 1], sk2[NG == 1 ? kMaxBlocks : 1], sk3[NG == 1 ? kMaxBlocks : 1];
  __shared__ int sflag[2];
  __shared__ int schunk[kEarlyMaxN / kRowChunk];     // hits per chunk of the winner's row, then their offsets
  __shared__ int stot;
  __shared__ int sj[kEarlyShare];                     // the block's share: target, old and new best cost,
  __shared__ float sbo[kEarlyShare], sbn[kEarlyShare];
  __shared__ double svs[kEarlyShare];                 // and its capacity scaled for fx_diff

  if (unfit(a)) return;
  const int S = *a.scale;
  for (int j = tid; j < a.ldt; j += kBlock) sball[j] = j < a.n ? a.c0 : -__builtin_inff();
  for (int i = tid; i < cnt; i += kBlock) ssel[i] = 0;
  init_gains(a, sG, lo, cnt, red);
  // Block 0 keeps the objective (in wave 1 after the start).
  long long L = 0;
  if (blk == 0) {
    const long long x = fx_capacity_part(a.v, a.n, a.c0, S);
    L = block_sum_i64(x, red);
  }
  auto publish = [&](int x) {
    if (NG == 1)
      publish_rows<true>(a, sG, ssel, lo, cnt, S, cand_slot(a.cand, x & 1, blk), epoch_of(x));
    else
      publish_argmax(sG, ssel, lo, cnt, S, cand_slot(a.cand, x & 1, blk), epoch_of(x), su);
  };
  publish(0);

  const int nch = a.ldt / kRowChunk;
  const int k_stop = a.k_end;                         // steps [0, k_stop) at most
  long long* mine = a.epart + size_t(blk) * a.ldp;
  int xc = 0;
  for (int step = 0; step < k_stop; ++step) {
    const unsigned long long* slots = cand_slot(a.cand, xc & 1, 0);
    const int tw = NG == 1 ? read_winner_rows<true>(a, slots, epoch_of(xc), nb, su, sflag, sk1, sk2, sk3)
                           : read_winner(slots, epoch_of(xc), nb, a.abort, a.poll_limit, su, sflag);
    ++xc;
    if (tw < 0) return;
    const int t = min(tw, a.n - 1);
    if (t >= lo && t < lo + cnt && tid == 0) {
      ssel[t - lo] = 1;
      a.selected[step] = t;
      if (a.step_gain) a.step_gain[step] = fx_to_double(sG[t - lo], S);
    }

    // The winner's row of T: every wave its chunks, all loads in flight.
    const f32x4* row = reinterpret_cast<const f32x4*>(a.T + size_t(t) * a.ldt);
    f32x4 xr[RL];
#pragma unroll
    for (int i = 0; i < RL; ++i)
      if (w + i * kWaves < nch) xr[i] = row[(w + i * kWaves) * (kRowChunk / 4) + lane];
    // Hits per chunk, their offsets in target order, and the total.
#pragma unroll
    for (int i = 0; i < RL; ++i) {
      const int q0 = w + i * kWaves;
      if (q0 < nch) {
        const f32x4 bo = *reinterpret_cast<const f32x4*>(sball + q0 * kRowChunk + 4 * lane);
        const f32x4 x = xr[i];
        const int c = __popcll(__ballot(x[0] < bo[0])) + __popcll(__ballot(x[1] < bo[1])) +
                      __popcll(__ballot(x[2] < bo[2])) + __popcll(__ballot(x[3] < bo[3]));
        if (lane == 0) schunk[q0] = c;
      }
    }
    __syncthreads();
    if (w == 0) {
      const int c0 = 2 * lane < nch ? schunk[2 * lane] : 0;
      const int c1 = 2 * lane + 1 < nch ? schunk[2 * lane + 1] : 0;
      const int incl = wave_scan_incl(c0 + c1);
      if (2 * lane < nch) schunk[2 * lane] = incl - c0 - c1;
      if (2 * lane + 1 < nch) schunk[2 * lane + 1] = incl - c1;
      if (lane == 63) stot = incl;
    }
    __syncthreads();
    const int H = stot;
    const int ns = a.eshares;                         // blocks that may take a share
    const int per = (H + ns - 1) / ns;                // at most ceil(n / ns) <= kEarlyShare
    const int e_lo = min(H, blk * per), e_hi = blk < ns ? min(H, e_lo + per) : e_lo;
    const int nshare = per > 0 ? (H + per - 1) / per : 0;   // blocks with a share
    // The block's share of the list; every target's new best cost; assign
    // for the own targets.
#pragma unroll
    for (int i = 0; i < RL; ++i) {
      const int q0 = w + i * kWaves;
      if (q0 < nch) {
        const int j0 = q0 * kRowChunk + 4 * lane;
        f32x4 bo = *reinterpret_cast<const f32x4*>(sball + j0);
        const f32x4 x = xr[i];
        int at = schunk[q0];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const bool hit = x[c] < bo[c];
          const unsigned long long mk = __ballot(hit);
          const int e = at + __popcll(mk & ((1ull << lane) - 1ull));
          if (hit) {
            const int j = j0 + c;
            if (e >= e_lo && e < e_hi) {
              sj[e - e_lo] = j;
              sbo[e - e_lo] = bo[c];
              sbn[e - e_lo] = x[c];
              svs[e - e_lo] = fx_scale(double(a.v[j]), S);
            }
            if (a.assign && unsigned(j - lo) < unsigned(cnt)) a.assign[j] = t;
            bo[c] = x[c];
          }
          at += __popcll(mk);
        }
        *reinterpret_cast<f32x4*>(sball + j0) = bo;
      }
    }
    __syncthreads();

    // The share's rows of the cost, in passes over kEarlyPass of the
    // thread's columns at a time, with the next kEarlyDepth rows' loads in
    // flight while a row is summed.  Loads past the share repeat its last
    // row and columns past n read column n - 1, so that every load is issued
    // unconditionally (the waits then count them exactly); such values are
    // never summed.
    const int nsh = e_hi - e_lo;
    if (nsh > 0) {
#pragma unroll 1
      for (int h = 0; h < kEarlyCols; h += kEarlyPass) {
        long long acc[kEarlyPass];
        float buf[kEarlyDepth][kEarlyPass];
#pragma unroll
        for (int q = 0; q < kEarlyPass; ++q) acc[q] = 0;
        auto load = [&](float* dst, int e) {
          const float* r = a.C + size_t(sj[min(e, nsh - 1)]) * a.n;
#pragma unroll
          for (int q = 0; q < kEarlyPass; ++q)
            dst[q] = __builtin_nontemporal_load(r + min(tid + kBlock * (h + q), a.n - 1));
        };
#pragma unroll
        for (int d = 0; d < kEarlyDepth; ++d) load(buf[d], d);
        for (int e = 0; e < nsh; e += kEarlyDepth) {
#pragma unroll
          for (int d = 0; d < kEarlyDepth; ++d) {
            float x[kEarlyPass];
#pragma unroll
            for (int q = 0; q < kEarlyPass; ++q) x[q] = buf[d][q];
            load(buf[d], e + d + kEarlyDepth);
            if (e + d < nsh) {
              const float bo = sbo[e + d], bn = sbn[e + d];
              const double vs = svs[e + d];
#pragma unroll
              for (int q = 0; q < kEarlyPass; ++q) {
                // A column that cost at least the old best contributes 0
                // before and after.
                if (tid + kBlock * (h + q) < a.n && x[q] < bo)
                  acc[q] += fx_diff(vs, fmaxf(bn - x[q], 0.f), bo - x[q]);
              }
            }
          }
        }
#pragma unroll
        for (int q = 0; q < kEarlyPass; ++q) {
          const int c = tid + kBlock * (h + q);
          if (c < a.n) put(reinterpret_cast<unsigned long long*>(mine + c), (unsigned long long)acc[q]);
        }
      }
      if (w == 0) {
        long long d = 0;
        for (int e = lane; e < nsh; e += 64) d += fx_diff(svs[e], sbn[e], sbo[e]);
        d = wave_sum_i64(d);
        if (lane == 0) put(reinterpret_cast<unsigned long long*>(mine + a.n), (unsigned long long)d);
      }
      __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's stores are done
    }
    __syncthreads();
    if (nsh > 0 && tid == 0) put(lens_slot(a.lens, blk), (unsigned long long)(step + 1));

    // Every share's sums, once its block has raised its flag for the step.
    if (tid == 0) sflag[0] = 0;
    __syncthreads();
    if (tid < nshare) {
      unsigned long long f;
      const unsigned long long want = (unsigned long long)(step + 1);
      if (!wait_slot(lens_slot(a.lens, tid), a.abort, a.poll_limit, [want](unsigned long long v) { return v == want; },
                     f))
        sflag[0] = 1;
    }
    __syncthreads();
    if (sflag[0]) return;
    {
      // All of a thread's loads are issued before any is used (a row past
      // nshare, or a column past cnt, is read from a valid address and not
      // summed).
      constexpr int kRead = 16;                       // loads in flight: two rounds for 256 blocks
#pragma unroll
      for (int q = 0; q < NG; ++q) {
        const int own = q * 64 + lane;
        const int col = min(lo + min(own, max(cnt - 1, 0)), a.n - 1);
        long long s = 0;
        for (int b0 = 0; b0 < nshare; b0 += kRead * kWaves) {
          unsigned long long x[kRead];
#pragma unroll
          for (int m = 0; m < kRead; ++m)
            x[m] = get(reinterpret_cast<const unsigned long long*>(
                a.epart + size_t(min(b0 + w + kWaves * m, ns - 1)) * a.ldp + col));
#pragma unroll
          for (int m = 0; m < kRead; ++m)
            if (own < cnt && b0 + w + kWaves * m < nshare) s += (long long)x[m];
        }
        red[q * kBlock + tid] = s;
      }
    }
    if (blk == 0 && w == 1) {
      constexpr int kRead = kMaxBlocks / 64;
      unsigned long long x[kRead];
#pragma unroll
      for (int m = 0; m < kRead; ++m)
        x[m] = get(reinterpret_cast<const unsigned long long*>(a.epart + size_t(min(lane + 64 * m, ns - 1)) * a.ldp + a.n));
      long long s = 0;
#pragma unroll
      for (int m = 0; m < kRead; ++m)
        if (lane + 64 * m < nshare) s += (long long)x[m];
      L += wave_sum_i64(s);
      if (lane == 0 && a.step_obj) a.step_obj[step] = fx_to_double(L, S);
    }
    __syncthreads();
    if (tid < 64) {
#pragma unroll
      for (int q = 0; q < NG; ++q)
        if (q * 64 + tid < cnt) {
          long long s = sG[q * 64 + tid];
#pragma unroll
          for (int r = 0; r < kWaves; ++r) s += red[q * kBlock + r * 64 + tid];
          sG[q * 64 + tid] = s;
        }
    }
    if (NG > 1) __syncthreads();
    // The next exchange's candidates (one column group: wave 0, which also
    // wrote the gains), unless this was the last step.
    if (step + 1 < a.k) publish(xc);
    if (step + 1 == k_stop || H < kEarlyMinHits) {
      // Hand over before step + 1.
      __syncthreads();
      for (int i = tid; i < cnt; i += kBlock) {
        a.ho_gain[lo + i] = sG[i];
        a.ho_sel[lo + i] = ssel[i];
      }
      if (blk == 0) {
        for (int j = tid; j < a.ldt; j += kBlock) a.ho_b[j] = sball[j];
        if (tid == 64) {
          a.ho_misc[0] = L;
          a.ho_misc[1] = xc;
          a.ho_misc[2] = step + 1;
        }
      }
      return;
    }
  }
}

template <int NG>
__global__ __launch_bounds__(kBlock) void sgs_early_kernel(IncDev a) { early_body<NG>(a, blockIdx.x, gridDim.x); }

// ---------------------------------------------------------------------------
// The rows schedule's later steps from candidate lists.
//
// Best costs only fall, so a pair (candidate c, target j) with C(c, j) >= b_j
// never changes a gain again.  After the first steps few pairs are left (at
// n = 6272: 229 per candidate on average after 8 picks, 60 after 64, 18 after
// 128).  The rows schedule then hands its state over (best costs, running
// gains, chosen flags, objective); list_build_kernel writes every candidate's
// pairs (target, cost) into a list, and sgs_list_kernel runs the remaining
// steps from the lists.
//
// A step needs the exchange of candidates only because the gains of other
// blocks' columns are not known.  The list kernel therefore takes many steps
// per exchange: a round.  Each block publishes its kPub best candidates with
// their exact gains; every block takes the same set of up to kSet best ones,
// and the largest gain left outside the set as the bound (all comparisons by
// gain_key, as in the exchanges of keys).  The lists of the
// set are then held in registers, and every block
// runs the greedy among them: the best of the set is the next pick as long as
// its gain is above the bound (gains only fall, so no candidate outside can
// catch up); its hits lower the best costs in LDS, the other candidates of the
// set sum their changes from their own entries whose best cost fell, and the
// block's own columns theirs from its pairs in LDS, indexed by target.  All
// terms are the fixed-point terms of the rows of T, so the picks are the same.
// A round takes about fourteen steps with kSet = 32 (nine with 16, six with 8;
// the prune of 6272 tokens takes 2.07 ms with 32, 2.15 with 16).
//
// Bound by instruction issue and LDS latency: about 1.5 us a step at n = 4096
// .. 16384, a round's exchange (poll 3 us, choosing the set 2 us, its lists
// 2.5 us, publishing 1.5 us) included; with a step or a chain of up to three
// predicted ones per exchange it took 2.1 to 2.8 us.  Two waves per SIMD
// (256 threads leave the latencies bare: 1.3 x the time; one wave per list
// and 1024 threads issue every uniform instruction four times per SIMD).
//
// A candidate with more pairs than a list holds keeps its row of T: it stays
// out of the set (its gain enters the bound) until it is the best of all, and
// is then picked alone, its hits read from that row.  A block whose own pairs
// do not fit in LDS reads the segments of the hits' rows of the cost over its
// own columns instead.
constexpr int kListCap = 512;                         // pairs a list holds at most
constexpr int kListBlock = 512;                       // threads of the list kernel: two waves per SIMD
constexpr int kListWaves = kListBlock / 64;
constexpr int kSet = 32;                              // candidates a round considers at most
constexpr int kChunksPer = 8;                        // chunks of 64 list entries a wave holds
constexpr int kSetChunks = kListWaves * kChunksPer;   // those of a set
constexpr int kPub = 4;                               // candidates a block publishes
constexpr int kPubWords = kPub + 3;                   // gains, indices, the best gain left out, list lengths
constexpr int kKeyLow = 16;                           // low bits of a gain_key that compare second
constexpr unsigned kKeyLowMask = (1u << kKeyLow) - 1u;
constexpr int kHitCap = 96;                          // hits a wave collects before it applies them
constexpr int kHitPick = kListCap / kListWaves;       // of one pick at most
static_assert(kHitPick % 64 == 0 && kHitPick < kHitCap, "a pick's chunks are spread evenly over the waves");
constexpr int kListMaxN = kRowChunk * kWaves * 8;     // 16384
constexpr int kListLds = 134 * 1024;                  // dynamic LDS of the list kernel at most

// The list kernel's LDS: gains and chosen flags of W columns, the best costs
// and (n <= kListLdsV: beyond it they would halve the room for the pairs) the
// capacities, the own pairs' first index per target (16 bits each, targets 0 .. n), their
// costs and candidates.
constexpr int kListLdsV = 8192;
__host__ __device__ __forceinline__ int list_off_words(int n) { return (n + 2) / 2; }
size_t list_lds_fixed(int64_t n, int W) {
  return size_t((W + 1) & ~1) * 8 + size_t(rows_ldt(n)) * 4 * (n <= kListLdsV ? 2 : 1) +
         size_t(list_off_words(int(n))) * 4 + size_t((W + 3) & ~3);
}
int list_ent(int64_t n, int W) { return int(std::min<size_t>(65535, (size_t(kListLds) - list_lds_fixed(n, W)) / 5)) & ~3; }

// One wave per candidate: its pairs from its row of T against the handed
// over best costs, gathered in LDS and then written as a whole (the list may
// lie at the start of the row itself).
__global__ __launch_bounds__(256) void list_build_kernel(IncDev a) {
  __shared__ uint2 sl[4][kListCap];
  if (*a.abort || unfit(a)) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c = blockIdx.x * 4 + w;
  if (c >= a.n) return;
  const f32x4* row = reinterpret_cast<const f32x4*>(a.T + size_t(c) * a.ldt);
  const f32x4* bb = reinterpret_cast<const f32x4*>(list_ho_b(a));
  const int nch = a.ldt / kRowChunk;
  const unsigned long long lt = (1ull << lane) - 1ull;
  int m = 0;
  for (int q0 = 0; q0 < nch; q0 += 8) {
    f32x4 x[8], b[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (q0 + u < nch) {
        x[u] = __builtin_nontemporal_load(row + (q0 + u) * (kRowChunk / 4) + lane);
        b[u] = bb[(q0 + u) * (kRowChunk / 4) + lane];
      }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (q0 + u >= nch) break;
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) {
        const bool hit = x[u][cc] < b[u][cc];         // never past n, where b = -inf
        const unsigned long long mk = __ballot(hit);
        if (hit) {
          const int pos = m + __popcll(mk & lt);
          if (pos < a.lcap) sl[w][pos] = uint2{unsigned((q0 + u) * kRowChunk + 4 * lane + cc), __float_as_uint(x[u][cc])};
        }
        m += __popcll(mk);
      }
    }
  }
  // The wave's own LDS writes are read back by the same wave.
  __builtin_amdgcn_wave_barrier();
  if (m <= a.lcap) {
    uint2* dst = a.lists + size_t(c) * a.lstride;
    for (int e = lane; e < m; e += 64) dst[e] = sl[w][e];
  }
  if (lane == 0) a.llen[c] = unsigned(m);
}

__device__ __forceinline__ int gain_bits(long long g) { return g < 0 ? -1 : __float_as_int(float(g)); }
__device__ __forceinline__ long long lane_i64(long long x, int l) { return (long long)lane_u64((unsigned long long)x, l); }

// The kPub first unchosen columns of the block in the order of candidates,
// and the gain of the next one, left out.  Every thread counts, for one column, the columns
// of its part that come before it (a maximum after another over one wave took
// four times as long); wave 0 publishes.  Words kListWord + r hold the gains,
// the next the own indices (8 bits each), then the rest's gain and the
// lists' lengths (12 bits each).  64 NG columns at most; starts and ends a
// phase between barriers of the whole block.
template <int NG>
__device__ __forceinline__ void publish_list(const IncDev& a, const unsigned long long* sG, const unsigned char* ssel,
                                             const unsigned short* slen, int lo, int cnt, int* srank, int* stop,
                                             unsigned long long* slot, unsigned long long epoch) {
  constexpr int kCols = 64 * NG, kParts = kListBlock / kCols;
  const int tid = threadIdx.x;
  const int i = tid % kCols, part = tid / kCols;
  if (tid < kPub + 1) stop[tid] = -1;
  {
    const int per = (cnt + kParts - 1) / kParts, m1 = min(cnt, (part + 1) * per);
    // Own columns from `bnd` on lie in the next group.  Chosen columns count
    // as gain -1 (key 0).
    const int bnd = (group_of(a, lo) + 1) * a.grp - lo;
    const long long g = i < cnt && !ssel[i] ? (long long)sG[i] : -1;
    int before = 0;
    if (bnd >= cnt) {
      for (int m = part * per; m < m1; ++m) {
        const long long x = ssel[m] ? -1 : (long long)sG[m];
        before += x + (m < i ? 1 : 0) > g ? 1 : 0;
      }
    } else {
      const unsigned long long u = gain_key(g);
      for (int m = part * per; m < m1; ++m) {
        const long long x = ssel[m] ? -1 : (long long)sG[m];
        const bool same = (m < bnd) == (i < bnd);
        before += (same ? x : (long long)gain_key(x)) + (m < i ? 1 : 0) > (same ? g : (long long)u) ? 1 : 0;
      }
    }
    // srank[i] was left at zero by the previous call.
    if (i < cnt && g >= 0) atomicAdd(&srank[i], before);
  }
  lds_barrier();
  if (tid < kCols) {
    if (i < cnt && !ssel[i]) {
      const int r = srank[i];
      if (r <= kPub) stop[r] = i;
    }
    srank[i] = 0;
  }
  if (NG > 1) lds_barrier();
  if (tid < 64) {
    // The five columns, read back by the wave that wrote them.
    int col[kPub + 1];
#pragma unroll
    for (int r = 0; r <= kPub; ++r) col[r] = stop[r];
    unsigned idx = 0;
    unsigned long long lens = 0;
#pragma unroll
    for (int r = 0; r < kPub; ++r)
      if (col[r] >= 0) {
        idx |= unsigned(col[r]) << (8 * r);
        lens |= (unsigned long long)min(int(slen[col[r]]), 4095) << (12 * r);
      }
    // Lane r < kPub a gain, then indices, the rest's gain, lengths.
    int c = -1;
#pragma unroll
    for (int r = 0; r < kPub; ++r)
      if (tid == r) c = col[r];
    if (tid == kPub + 1) c = col[kPub];
    unsigned long long word = c >= 0 ? sG[max(c, 0)] : kNoGain;
    if (tid == kPub) word = idx;
    if (tid == kPub + 2) word = lens;
    if (tid < kPubWords) put(slot + kListWord + tid, word | epoch);
  }
}

// Steps k_begin .. k - 1 of a scene from the lists, by block `blk` of the
// scene's `nb` blocks (NG columns per lane: W <= 64 NG).
template <int NG>
__device__ __forceinline__ void list_body(const IncDev& a, int blk, int nb) {
  if (*a.abort || a.k_begin >= a.k || unfit(a)) return;
  extern __shared__ unsigned long long smem[];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lo = blk * a.W;
  const int cnt = max(0, min(a.n, lo + a.W) - lo);
  unsigned long long* sG = smem;                                   // [W] running gains (W rounded up to even)
  float* sball = reinterpret_cast<float*>(sG + ((a.W + 1) & ~1));  // [ldt] best costs
  // The block's own pairs by target: pairs [off(j), off(j + 1)) have target
  // j, each with its cost and its candidate (own index); off as 16-bit
  // values, two to a word.
  const bool v_lds = a.n <= kListLdsV;
  float* sv = sball + a.ldt;                                       // [ldt] capacities (v_lds)
  unsigned int* soffw = reinterpret_cast<unsigned int*>(v_lds ? sv + a.ldt : sv);
  unsigned char* ssel = reinterpret_cast<unsigned char*>(soffw + list_off_words(a.n));   // [W] chosen
  float* spc = reinterpret_cast<float*>(ssel + ((a.W + 3) & ~3));  // [lent]
  unsigned char* spk = reinterpret_cast<unsigned char*>(spc + a.lent);    // [lent]
  auto off = [&](int j) { return int((soffw[j >> 1] >> ((j & 1) * 16)) & 0xffffu); };
  __shared__ int soff[64 * NG + 1];                                 // each own candidate's first listed pair
  __shared__ int swt[kListWaves];
  // What a round reads from the exchange, and then, in the same memory, the
  // hits and changes its waves list.
  struct Exchange {
    unsigned long long gain[kPub + 1][kMaxBlocks];                  // gains, best gain left out
    unsigned long long len[kMaxBlocks];                             // list lengths
    int bits[kPub][kMaxBlocks];                                     // gain_bits of the gains
    unsigned idx[kMaxBlocks];                                       // indices
  };
  struct Picks {
    uint4 hit[kListWaves][kHitCap];                                 // target | pick << 16, new, old cost, capacity
    uint4 chg[kListWaves][64];                                      // a wave's changes: cost, new, old best, capacity
    int chm[kListWaves][64];                                        // and member
  };
  __shared__ union Round {
    Exchange x;
    Picks p;
  } sr;
  auto& sgw = sr.x.gain;
  auto& sgl = sr.x.len;
  auto& sgf = sr.x.bits;
  auto& sgi = sr.x.idx;
  auto& shit = sr.p.hit;
  auto& schg = sr.p.chg;
  auto& schm = sr.p.chm;
  __shared__ unsigned long long sset[kSet];                         // the set's gains
  __shared__ int sidx[kSet], slist[kSet];                           // indices and list lengths
  __shared__ long long sbound[4];
  __shared__ int sflag, stotal;
  __shared__ int spt[kSet];                                         // the round's picks
  __shared__ long long spg[kSet];                                   // their gains
  __shared__ unsigned long long sobj[kSet];                         // and changes of the objective (block 0)
  __shared__ unsigned long long sL;                                 // objective (block 0)
  __shared__ int srank[64 * NG], stop5[kPub + 1];                   // publish_list's
  __shared__ unsigned short slen[64 * NG];                          // own candidates' pairs, 65535 for more
  const int S = *a.scale;

  const float* hb = list_ho_b(a);
  for (int j = tid; j < a.ldt; j += kListBlock) {
    sball[j] = hb[j];
    if (v_lds) sv[j] = j < a.n ? a.v[j] : 0.f;
  }
  for (int i = tid; i < list_off_words(a.n); i += kListBlock) soffw[i] = 0u;
  if (tid < kSet) sobj[tid] = 0ull;
  if (tid < 64 * NG) srank[tid] = 0;
  if (tid == 0) {
    sflag = 0;
    sL = (unsigned long long)(blk == 0 ? a.ho_misc[0] : 0);
  }
  // Own candidates' pair counts: all of them (do they fit?) and the listed ones.
  if (w == 0) {
    int run = 0, all = 0;
    for (int q = 0; q < NG; ++q) {
      const int i = q * 64 + lane;
      const int m = i < cnt ? int(a.llen[lo + i]) : 0;
      const bool lng = m > a.lcap;
      if (i < cnt) {
        ssel[i] = a.ho_sel[lo + i];
        slen[i] = (unsigned short)min(m, 65535);
        sG[i] = (unsigned long long)a.ho_gain[lo + i];
      }
      const int incl = wave_scan_incl(lng ? 0 : m);
      soff[i + 1] = run + incl;
      run += __builtin_amdgcn_readlane(incl, 63);
      all += __builtin_amdgcn_readlane(wave_scan_incl(m), 63);
    }
    if (lane == 0) {
      soff[0] = 0;
      stotal = all;
    }
  }
  __syncthreads();
  const bool own_lds = stotal <= a.lent;                            // uniform over the block
  if (own_lds) {
    // Pairs per target (16-bit counts, two to a word), their inclusive
    // prefix over the targets, then each pair placed at its target's end,
    // which moves down to the target's first pair.  A long candidate's pairs
    // come from its row of T.
    const int npairs = soff[64 * NG];
    auto each_pair = [&](auto f) {
      for (int p0 = 0; p0 < npairs; p0 += 8 * kListBlock) {
        uint2 ev[8];
        int ci[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int pq = min(p0 + q * kListBlock + tid, npairs - 1);
          int c = 0;
#pragma unroll
          for (int st = 32 * NG; st > 0; st >>= 1)
            if (c + st < 64 * NG && soff[c + st] <= pq) c += st;
          ci[q] = c;
          ev[q] = a.lists[size_t(lo + c) * a.lstride + (pq - soff[c])];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
          if (p0 + q * kListBlock + tid < npairs) f(min(int(ev[q].x), a.n - 1), __uint_as_float(ev[q].y), ci[q]);
      }
      for (int i = 0; i < cnt; ++i)
        if (int(slen[i]) > a.lcap)
          for (int j = tid; j < a.n; j += kListBlock) {
            const float x = a.T[size_t(lo + i) * a.ldt + j];
            if (x < sball[j]) f(j, x, i);
          }
    };
    each_pair([&](int j, float, int) { atomicAdd(&soffw[j >> 1], 1u << ((j & 1) * 16)); });
    __syncthreads();
    const int per = (list_off_words(a.n) + kListBlock - 1) / kListBlock;   // words a thread scans
    const int w0 = min(tid * per, list_off_words(a.n)), w1 = min(w0 + per, list_off_words(a.n));
    int sum = 0;
    for (int i = w0; i < w1; ++i) sum += int(soffw[i] & 0xffffu) + int(soffw[i] >> 16);
    const int incl = wave_scan_incl(sum);
    if (lane == 63) swt[w] = incl;
    __syncthreads();
    int run = incl - sum;
#pragma unroll
    for (int q = 0; q < kListWaves; ++q)
      if (q < w) run += swt[q];
    for (int i = w0; i < w1; ++i) {
      const unsigned int wv = soffw[i];
      const int lo16 = run + int(wv & 0xffffu);
      const int hi16 = lo16 + int(wv >> 16);
      soffw[i] = unsigned(lo16) | (unsigned(hi16) << 16);
      run = hi16;
    }
    __syncthreads();
    each_pair([&](int j, float x, int i) {
      const unsigned int sh = (j & 1) * 16;
      const int pos = int((atomicSub(&soffw[j >> 1], 1u << sh) >> sh) & 0xffffu) - 1;
      spc[pos] = x;
      spk[pos] = (unsigned char)i;
    });
    __syncthreads();
  }

  // The own columns' changes of a wave's hits (a lane each, where ok) when
  // the pairs are not in LDS: the hits' rows of the cost, eight at a time.
  auto own_segments = [&](bool ok, int j, float x, float bo, double vs) {
    unsigned long long mk = __ballot(ok);
    const long long vb = __double_as_longlong(vs);
    long long g[NG];
#pragma unroll
    for (int q = 0; q < NG; ++q) g[q] = 0;
    while (mk) {
      int ln[8];
      float cv[8][NG];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        ln[u] = mk ? __builtin_ctzll(mk) : -1;
        mk = mk ? mk & (mk - 1) : 0ull;
        const int jr = __builtin_amdgcn_readlane(j, max(ln[u], 0));
#pragma unroll
        for (int q = 0; q < NG; ++q)
          cv[u][q] = (ln[u] >= 0 && q * 64 + lane < cnt) ? a.C[size_t(jr) * a.n + lo + q * 64 + lane] : __builtin_inff();
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int l = max(ln[u], 0);
        const float bor = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bo), l));
        const float xr = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
        const double vr = __longlong_as_double(
            (long long)(((unsigned long long)(unsigned)__builtin_amdgcn_readlane(int(vb >> 32), l) << 32) |
                        (unsigned)__builtin_amdgcn_readlane(int(vb), l)));
#pragma unroll
        for (int q = 0; q < NG; ++q)
          if (cv[u][q] < bor) g[q] += fx_diff(vr, fmaxf(xr - cv[u][q], 0.f), bor - cv[u][q]);
      }
    }
#pragma unroll
    for (int q = 0; q < NG; ++q)
      if (g[q] != 0) atomicAdd(&sG[q * 64 + lane], (unsigned long long)g[q]);
  };
  // A wave's hits, one a lane (where ok): at its pick (the round's ord-th)
  // target j fell from bo to x; v is its capacity.  The own columns' gains and
  // (block 0) the objective.
  auto apply_hits = [&](bool ok, int ord, int j, float x, float bo, float v) {
    const double vs = fx_scale(double(v), S);
    if (ok && own_lds) {
      const int p1 = off(j + 1);
      for (int p = off(j); p < p1; ++p) {
        const float cv = spc[p];
        if (cv < bo) atomicAdd(&sG[spk[p]], (unsigned long long)fx_diff(vs, fmaxf(x - cv, 0.f), bo - cv));
      }
    }
    if (!own_lds) own_segments(ok, j, x, bo, vs);
    if (blk == 0 && ok) atomicAdd(&sobj[ord], (unsigned long long)fx_diff(vs, x, bo));
  };

  // Hits a wave has listed: their consequences, and the assignment of the own
  // targets (by the last pick that lowered each: the one whose cost stands).
  auto flush = [&](int nh) {
    for (int e0 = 0; e0 < nh; e0 += 64) {
      const bool ok = e0 + lane < nh;
      const uint4 h = shit[w][ok ? e0 + lane : 0];
      const int j = int(h.x & 0xffffu), ord = int(h.x >> 16);
      const float x = __uint_as_float(h.y);
      apply_hits(ok, ord, j, x, __uint_as_float(h.z), __uint_as_float(h.w));
      if (ok && a.assign && unsigned(j - lo) < unsigned(cnt) && sball[j] == x) a.assign[j] = spt[ord];
    }
  };

  int step = a.k_begin;
  int gap = 1 << 20;                                                // the last round's threshold below its best
  publish_list<NG>(a, sG, ssel, slen, lo, cnt, srank, stop5, cand_slot(a.cand, 0, blk), epoch_of(0));
  for (int xc = 0; step < a.k; ++xc) {
    // The exchange: a wave reads eight slots per load, eight lanes each.
    {
      const unsigned long long ep = epoch_of(xc);
      const unsigned long long* slots = cand_slot(a.cand, xc & 1, 0) + kListWord;
      constexpr int kRead = kMaxBlocks / (8 * kListWaves);          // loads in flight: 4
      const int r = lane & 7;
      unsigned long long x[kRead];
      bool need[kRead];
#pragma unroll
      for (int q = 0; q < kRead; ++q) {
        need[q] = r < kPubWords && (w * kRead + q) * 8 + (lane >> 3) < nb;
        x[q] = ~ep;
      }
      for (unsigned int spins = 0;; ++spins) {
        bool miss = false;
#pragma unroll
        for (int q = 0; q < kRead; ++q)
          if (need[q] && (x[q] & kEpoch) != ep)
            x[q] = get(slots + size_t((w * kRead + q) * 8 + (lane >> 3)) * kSlotStride + r);
#pragma unroll
        for (int q = 0; q < kRead; ++q) miss = miss || (need[q] && (x[q] & kEpoch) != ep);
        if (!__ballot(miss)) break;
        if (__ballot(give_up(spins, a.poll_limit, a.abort))) {
          if (lane == 0) sflag = 1;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
#pragma unroll
      for (int q = 0; q < kRead; ++q)
        if (r < kPubWords) {
          // Blocks past nb publish nothing.
          const int b = (w * kRead + q) * 8 + (lane >> 3);
          x[q] = need[q] ? x[q] & ~kEpoch : (r == kPub || r == kPub + 2) ? 0ull : kNoGain;
          if (r < kPub) {
            sgw[r][b] = x[q];
            sgf[r][b] = gain_bits(word_gain(x[q]));
          } else if (r == kPub) {
            sgi[b] = unsigned(x[q]);
          } else if (r == kPub + 1) {
            sgw[kPub][b] = x[q];
          } else {
            sgl[b] = x[q];
          }
        }
    }
    lds_barrier();
    if (sflag) break;
    // The set: the candidates above a float threshold, found by bisection on
    // the blocks' best ones (the same in every wave) so that at most kSet lie
    // above it and their lists fit; wave w enters those of blocks 64 w ..
    // 64 w + 63.  One without a list stays out.
    int ns = 0;
    {
      int f[kPub][4], nc[kPub][4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const unsigned long long ln = sgl[lane + 64 * q];
#pragma unroll
        for (int r = 0; r < kPub; ++r) {
          const int l = int(ln >> (12 * r)) & 0xfff;
          f[r][q] = l > a.lcap ? -1 : sgf[r][lane + 64 * q];
          nc[r][q] = max(1, (l + 63) >> 6);
        }
      }
      const int ob = (w & 3) * 64 + lane;
      unsigned long long og[kPub + 1];
#pragma unroll
      for (int r = 0; r <= kPub; ++r) og[r] = sgw[r][ob];
      const unsigned oi = sgi[ob];
      const unsigned long long ol = sgl[ob];
      const int M = int(wave_max_u32(unsigned(max(max(f[0][0], f[0][1]), max(f[0][2], f[0][3])) + 1))) - 1;
      auto count1 = [&](int T) {
        int c = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) c += __popcll(__ballot(f[0][q] > T));
        return c;
      };
      constexpr int kLow = kSet * 5 / 8, kHigh = kSet - 2;          // of the blocks' best ones
      int lo_t = -1, hi_t = M, T = max(-1, M - gap);
      bool low = false;                                             // count1(lo_t) is known to be too many
      for (int it = 0; it < 64; ++it) {
        const int c = count1(T);
        if (c > kHigh) {
          lo_t = T;
          low = true;
        } else if (c < kLow && T > -1) {
          hi_t = T;
        } else {
          break;
        }
        if (hi_t - lo_t <= 1) {
          T = hi_t;
          break;
        }
        // Without a lower end yet: twice as far below the best.
        T = low ? lo_t + (hi_t - lo_t) / 2 : M - T > (1 << 28) ? -1 : max(-1, M - 2 * (M - T));
      }
      gap = max(1, M - T);
      int base = 0;                                                 // members of the waves before
      for (;;) {
        ns = base = 0;
        int ch = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (q == w) base = ns;
#pragma unroll
          for (int r = 0; r < kPub; ++r) {
            ns += __popcll(__ballot(f[r][q] > T));
            ch += f[r][q] > T ? nc[r][q] : 0;
          }
        }
        if (ns <= kSet && wave_sum_i32(ch) <= kSetChunks) break;
        T += (M - T + 1) / 2;                                       // none lies above M
      }
      if (w < 4) {
        long long bound = word_gain(og[kPub]);
#pragma unroll
        for (int r = 0; r < kPub; ++r) {
          const long long g = word_gain(og[r]);
          const int l = int(ol >> (12 * r)) & 0xfff;
          const bool in = l <= a.lcap && sgf[r][ob] > T;
          const unsigned long long mk = __ballot(in);
          if (in) {
            const int at = base + __popcll(mk & ((1ull << lane) - 1ull));
            sset[at] = (unsigned long long)g;
            sidx[at] = min(ob * a.W + int((oi >> (8 * r)) & 0xffu), a.n - 1);
            slist[at] = l;
          } else {
            bound = max(bound, g);
          }
          base += __popcll(mk);
        }
        bound = (long long)wave_max_u64((unsigned long long)(bound + 1)) - 1;
        if (lane == 0) sbound[w] = bound;
      }
    }
    lds_barrier();
    long long bound = sbound[0];
#pragma unroll
    for (int q = 1; q < 4; ++q) bound = max(bound, sbound[q]);
    const unsigned long long bkey = gain_key(bound);
    int np = 0;                                                     // picks of the round
    {
      // The set's lists in chunks of 64 entries, member after member: chunk c
      // in wave c mod kListWaves.  Target, cost, capacity and the target's best cost
      // as last seen; lane m < ns looks after member m.
      const bool mine = lane < ns;
      const int myidx = mine ? sidx[lane & (kSet - 1)] : INT_MAX;
      const int mylen = mine ? slist[lane & (kSet - 1)] : 0;
      const int mygrp = group_of(a, myidx);
      const int mych = (mylen + 63) >> 6;
      const int myend = wave_scan_incl(mych), mystart = myend - mych;
      const int nch = __builtin_amdgcn_readlane(myend, 63);
      int mem[kChunksPer];                                          // uniform
      int ej[kChunksPer];
      float ec[kChunksPer], eb[kChunksPer], ev[kChunksPer];
      {
        uint2 en[kChunksPer];
        int left[kChunksPer];
#pragma unroll
        for (int i = 0; i < kChunksPer; ++i) {
          const int c = i * kListWaves + w;
          mem[i] = -1;
          if (c >= nch) continue;
          const int m = __builtin_ctzll(__ballot(myend > c));
          const int o = (c - __builtin_amdgcn_readlane(mystart, m)) * 64;
          const uint2* l = a.lists + size_t(__builtin_amdgcn_readlane(myidx, m)) * a.lstride + o;
          left[i] = __builtin_amdgcn_readlane(mylen, m) - o;
          mem[i] = m;
          en[i] = l[min(lane, left[i] - 1)];
        }
#pragma unroll
        for (int i = 0; i < kChunksPer; ++i) {
          ej[i] = 0;
          ec[i] = __builtin_inff();
          ev[i] = 0.f;
          eb[i] = -__builtin_inff();
          if (i * kListWaves + w >= nch) continue;
          if (lane < left[i]) {
            ej[i] = min(int(en[i].x), a.n - 1);
            ec[i] = __uint_as_float(en[i].y);
          }
          ev[i] = v_lds ? sv[ej[i]] : a.v[ej[i]];
          eb[i] = sball[ej[i]];
        }
      }
      unsigned done = 0;                                            // members picked
      int nh = 0;                                                   // hits this wave has listed
      lds_barrier();   // every wave has read the best costs before the first pick lowers any
      for (;; ++np) {
        // The first of the set, the same in every wave: the largest high word
        // of the keys, then (rarely) the low word, then first_of.
        const long long gl = mine && !((done >> (lane & 31)) & 1u) ? (long long)sset[lane & (kSet - 1)] : -1;
        const unsigned long long u = gain_key(gl);
        const unsigned hm = half_max_u32(unsigned(u >> kKeyLow));
        unsigned long long tie = __ballot(unsigned(u >> kKeyLow) == hm) & ((1ull << kSet) - 1ull);
        if (__popcll(tie) > 1) {
          const unsigned lm = half_max_u32(unsigned(u >> kKeyLow) == hm ? unsigned(u) & kKeyLowMask : 0u);
          tie &= __ballot((unsigned(u) & kKeyLowMask) == lm);
          if (__popcll(tie) > 1) {
            if (((tie >> lane) & 1ull) && gl != lane_i64(gl, __builtin_ctzll(tie))) note_tie(a);
            tie = 1ull << first_of(tie, mygrp, gl, myidx);
          }
        }
        const int slot = __builtin_ctzll(tie);
        const long long g = lane_i64(gl, slot);
        // (The first one has to beat the bound too: it may not when the best
        // of all has no list, or too many share its float gain.)
        if (step + np >= a.k || g < 0 || lane_u64(u, slot) <= bkey) break;
        if (tid == 0) {
          spt[np] = __builtin_amdgcn_readlane(myidx, slot);
          spg[np] = g;
        }
        // The pick's hits, listed by the waves that hold its chunks.
        if (nh > kHitCap - kHitPick) {
          flush(nh);
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");   // its assignments come before later ones
          nh = 0;
        }
#pragma unroll
        for (int i = 0; i < kChunksPer; ++i) {
          if (i * kListWaves + w >= nch) break;
          if (mem[i] != slot) continue;                             // uniform
          const int j = ej[i];
          const float x = ec[i], bo = sball[j];
          const bool ok = x < bo;
          const unsigned long long mk = __ballot(ok);
          if (ok) {
            sball[j] = x;
            shit[w][nh + __popcll(mk & ((1ull << lane) - 1ull))] =
                uint4{unsigned(j) | (unsigned(np) << 16), __float_as_uint(x), __float_as_uint(bo),
                      __float_as_uint(ev[i])};
          }
          nh += __popcll(mk);
        }
        done |= 1u << slot;
        lds_barrier();
        // The members' changes, from the entries whose best cost fell (the
        // first chunks' best costs are read together).
        float bn[kChunksPer];
#pragma unroll
        for (int i = 0; i < kChunksPer; ++i)
          if (i < 4 || i * kListWaves + w < nch) bn[i] = sball[ej[i]];
        // Few entries change in a chunk, so they are gathered first.
        int nc = 0;
        auto settle = [&]() {
          const bool ok = lane < nc;
          const uint4 h = schg[w][lane];
          if (ok) {
            const float cv = __uint_as_float(h.x), n1 = __uint_as_float(h.y), o1 = __uint_as_float(h.z);
            atomicAdd(&sset[schm[w][lane]], (unsigned long long)fx_diff(fx_scale(double(__uint_as_float(h.w)), S),
                                                                        fmaxf(n1 - cv, 0.f), o1 - cv));
          }
          nc = 0;
        };
#pragma unroll
        for (int i = 0; i < kChunksPer; ++i) {
          if (i * kListWaves + w >= nch) break;
          const bool fell = bn[i] < eb[i];
          const unsigned long long mk = __ballot(fell && ec[i] < eb[i]);
          if (mk) {
            const int m = __popcll(mk);
            if (nc + m > 64) settle();
            if ((mk >> lane) & 1ull) {
              const int at = nc + __popcll(mk & ((1ull << lane) - 1ull));
              schg[w][at] = uint4{__float_as_uint(ec[i]), __float_as_uint(bn[i]), __float_as_uint(eb[i]),
                                  __float_as_uint(ev[i])};
              schm[w][at] = mem[i];
            }
            nc += m;
            eb[i] = fminf(eb[i], bn[i]);
          }
        }
        if (nc) settle();
        lds_barrier();
      }
      flush(nh);
    }
    if (np == 0) {
      // The best candidate of all, alone, from its list or its row of T.  Once
      // its gain is zero all are, and stay so: the smallest indices follow, as
      // many as its block published (600 picks of 6000 tokens, all but one of
      // no gain: 5.25 ms with one a round, 1.84 so, 3.14 in the rows kernel).
      unsigned long long kb[4], kmax = 0ull;
      int ib[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int b = lane + 64 * q;
        kb[q] = gain_key(word_gain(sgw[0][b]));
        ib[q] = b * a.W + int(sgi[b] & 0xffu);
        kmax = max(kmax, kb[q]);
      }
      const unsigned long long top = wave_max_u64(kmax);
      if (top == 0ull) break;                                       // never with a candidate left
      // Of the blocks' best ones with that key: the lowest group's (it holds
      // the smallest index), there the largest gain, then the smallest index.
      int im = INT_MAX;
#pragma unroll
      for (int q = 0; q < 4; ++q) im = min(im, kb[q] == top ? ib[q] : INT_MAX);
      const int gm = group_of(a, wave_min_i32(im));
      long long gx = -1;
      int bx = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {                                 // increasing index
        const long long gq = word_gain(sgw[0][lane + 64 * q]);
        if (kb[q] == top && group_of(a, ib[q]) == gm && gq > gx) {
          gx = gq;
          bx = lane + 64 * q;
        }
      }
      const unsigned long long gt = wave_max_u64((unsigned long long)(gx + 1));
      const int wb = wave_min_i32((unsigned long long)(gx + 1) == gt ? bx : INT_MAX);
      const long long gb = word_gain(sgw[0][wb]);
      np = 1;
      if (gb == 0) {
#pragma unroll
        for (int r = 1; r < kPub; ++r)
          if (np == r && word_gain(sgw[r][wb]) == 0) np = r + 1;
        np = min(np, a.k - step);
      }
      if (w == 0 && (a.abort_init & 2u)) {
#pragma unroll
        for (int r = 0; r <= kPub; ++r)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const long long gq = word_gain(sgw[r][lane + 64 * q]);
            if (gq != gb && gain_key(gq) == top) note_tie(a);
          }
      }
      np = __builtin_amdgcn_readfirstlane(np);
      for (int i = 0; i < np; ++i) {
        const int t = min(__builtin_amdgcn_readfirstlane(wb * a.W + int((sgi[wb] >> (8 * i)) & 0xffu)), a.n - 1);
        const int len = __builtin_amdgcn_readfirstlane(int(sgl[wb] >> (12 * i)) & 0xfff);
        const bool listed = len <= a.lcap;
        // Every wave has read the best costs, and the assignments of the pick
        // before come before this one's.
        __syncthreads();
        for (int e0 = w * 64; e0 < (listed ? len : a.n); e0 += kListBlock) {
          const int e = e0 + lane;
          int j = 0;
          float x = __builtin_inff();
          if (listed && e < len) {
            const uint2 en = a.lists[size_t(t) * a.lstride + e];
            j = min(int(en.x), a.n - 1);
            x = __uint_as_float(en.y);
          } else if (!listed && e < a.n) {
            j = e;
            x = a.T[size_t(t) * a.ldt + j];
          }
          const float bo = sball[j];
          const bool ok = x < bo;
          if (!__ballot(ok)) continue;
          if (ok) {
            sball[j] = x;
            if (a.assign && unsigned(j - lo) < unsigned(cnt)) a.assign[j] = t;
          }
          apply_hits(ok, i, j, x, bo, ok ? a.v[j] : 0.f);
        }
        if (tid == 0) {
          spt[i] = t;
          spg[i] = gb;
        }
      }
      lds_barrier();
    }
    // The round's picks: chosen flags, and (block 0) the outputs.
    if (w == 0) {
      if (lane < np) {
        const int t = spt[lane];
        if (t >= lo && t < lo + cnt) ssel[t - lo] = 1;
      }
    }
    __syncthreads();
    if (step + np < a.k)
      publish_list<NG>(a, sG, ssel, slen, lo, cnt, srank, stop5, cand_slot(a.cand, (xc + 1) & 1, blk), epoch_of(xc + 1));
    if (w == 1 && blk == 0) {
      unsigned long long L = sL;
      for (int i = 0; i < np; ++i) L += lane >= i ? sobj[i] : 0ull;
      if (lane < np) {
        a.selected[step + lane] = spt[lane];
        if (a.step_gain) a.step_gain[step + lane] = fx_to_double(spg[lane], S);
        if (a.step_obj) a.step_obj[step + lane] = fx_to_double((long long)L, S);
      }
      if (lane < kSet) sobj[lane] = 0ull;
      if (lane == np - 1) sL = L;
    }
    step += np;
  }
}

template <int NG>
__global__ __launch_bounds__(kListBlock) void sgs_list_kernel(IncDev a) { list_body<NG>(a, blockIdx.x, gridDim.x); }

// The fixed-point scale of a scene (one block; the sum in the same order as
// every block of the greedy would take it).
__global__ __launch_bounds__(kBlock) void inc_scale_kernel(IncDev a, int* scale) {
  __shared__ double sd[kWaves];
  const int S = fixed_scale(a, sd);
  if (threadIdx.x == 0) *scale = S;
  if (a.abort_init & 2u) {
    // Capacities the fixed point does not hold: negative, infinite or NaN.
    bool bad = false;
    for (int j = threadIdx.x; j < a.n; j += kBlock) bad = bad || !(a.v[j] >= 0.f && a.v[j] < __builtin_inff());
    if (bad) atomicOr(a.abort + kUnfitWord, 1u);
  }
}

// Step-0 gains, every row at b = c0, split over a grid of (column strip,
// row range) blocks so that the pass runs with many more waves in flight than
// the greedy's one block per compute unit: block (b, p) sums rows
// [p R, (p + 1) R) of columns [64 b, 64 b + 64) into part[p][column], 64-bit
// fixed point, four waves adding in wave order.  A round covers 64 rows, 16
// per wave.  With WT the round's 64 x 64 tile also goes to T through LDS:
// lane `col` of a wave holds C_tm[j0 .. j0 + 16)[col], i.e. a piece of row
// `col` of T; after a barrier each store instruction writes four rows of T,
// 256 contiguous bytes each (16 lanes of 16 bytes), so every line written is
// whole.  R is a multiple of 16 and rows of T are only written below the
// range's end (n, padding aside, for the last range).
constexpr int kPassThreads = 256;
constexpr int kPassWaves = kPassThreads / 64;
constexpr int kPassRows = 16;
constexpr int kPassCols = 64;                       // whatever W the greedy has: a lane a column
constexpr int kPassTile = kPassWaves * kPassRows;   // rows per round
constexpr int kPassLd = kPassTile + 4;               // LDS row of the tile: 16-byte aligned, banks spread

__host__ __device__ __forceinline__ int pass_rows(int n, int P) {
  return ((n + P - 1) / P + kPassRows - 1) / kPassRows * kPassRows;
}

template <bool WT, bool CHECK>
__global__ __launch_bounds__(kPassThreads) void inc_first_pass_kernel(IncDev a, long long* part) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lo = blockIdx.x * kPassCols, cnt = min(a.n - lo, kPassCols);
  const int R = pass_rows(a.n, a.P), r0 = blockIdx.y * R, r1 = min(a.n, r0 + R);
  const int S = *a.scale;
  __shared__ long long red[kPassThreads];
  __shared__ __attribute__((aligned(16))) float tile[WT ? 64 : 1][WT ? kPassLd : 1];   // [column][row of the round]
  for (int cc = 0; cc < cnt; cc += 64) {
    const bool colok = cc + lane < cnt;
    const int col = lo + cc + lane;
    // The next round's loads are issued before the current round's terms
    // are formed; two accumulators.
    long long g0 = 0, g1 = 0;
    bool bad = false;
    float xn[kPassRows], vn[kPassRows];
    auto load = [&](int j0) {
#pragma unroll
      for (int u = 0; u < kPassRows; ++u) {
        const int j = j0 + u;
        xn[u] = (colok && j < r1) ? __builtin_nontemporal_load(a.C + size_t(j) * a.n + col) : a.c0;
        vn[u] = j < r1 ? a.v[j] : 0.f;
      }
    };
    load(r0 + w * kPassRows);
    for (int jr = r0; jr < r1; jr += kPassTile) {   // uniform over the block
      const int j0 = jr + w * kPassRows;
      float x[kPassRows], vj[kPassRows];
#pragma unroll
      for (int u = 0; u < kPassRows; ++u) {
        x[u] = xn[u];
        vj[u] = vn[u];
        if (CHECK) bad = bad || !(x[u] >= 0.f);
      }
      if (jr + kPassTile < r1) load(j0 + kPassTile);   // rows past r1 load as zero terms
#pragma unroll
      for (int u = 0; u < kPassRows; u += 2) {
        g0 += fx(double(vj[u]) * double(fmaxf(a.c0 - x[u], 0.f)), S);
        g1 += fx(double(vj[u + 1]) * double(fmaxf(a.c0 - x[u + 1], 0.f)), S);
      }
      if (WT) {
#pragma unroll
        for (int q = 0; q < kPassRows / 4; ++q)
          *reinterpret_cast<f32x4*>(&tile[lane][w * kPassRows + 4 * q]) =
              f32x4{x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]};
        __syncthreads();
        // Instruction q: columns 16 q .. 16 q + 15, lane piece (tid % 16) of
        // four rows; a piece starting below r1 lies below ldt.
#pragma unroll
        for (int q = 0; q < 64 / (kPassThreads / 16); ++q) {
          const int c = q * (kPassThreads / 16) + tid / 16, r = (tid % 16) * 4;
          if (cc + c < cnt && jr + r < r1)
            *reinterpret_cast<f32x4*>(a.T + size_t(lo + cc + c) * a.ldt + jr + r) =
                *reinterpret_cast<const f32x4*>(&tile[c][r]);
        }
        __syncthreads();
      }
    }
    if (CHECK && __ballot(bad) && lane == 0) atomicOr(a.abort + kUnfitWord, 1u);
    red[tid] = g0 + g1;
    __syncthreads();
    if (tid < 64 && cc + tid < cnt) {
      long long s = 0;
#pragma unroll
      for (int q = 0; q < kPassWaves; ++q) s += red[q * 64 + tid];
      part[size_t(blockIdx.y) * a.n + lo + cc + tid] = s;
    }
    __syncthreads();
  }
}

// Several scenes in one launch: scene s runs on blocks [g0[s], g0[s + 1])
// with its own slots, change lists and abort flag, so the scenes' greedies
// proceed independently side by side.
constexpr int kMaxBatch = 16;

struct IncBatch {
  int count;
  int g0[kMaxBatch + 1];
  IncDev scene[kMaxBatch];
};
static_assert(sizeof(IncBatch) <= 4096, "kernel arguments");

__global__ __launch_bounds__(kBlock) void sgs_inc_batch_kernel(IncBatch b) {
  int s = 0;
  while (s + 1 < b.count && int(blockIdx.x) >= b.g0[s + 1]) ++s;
  inc_body(b.scene[s], int(blockIdx.x) - b.g0[s], b.g0[s + 1] - b.g0[s]);
}

template <int NG, int RL>
__global__ __launch_bounds__(kBlock) void sgs_rows_batch_kernel(IncBatch b) {
  int s = 0;
  while (s + 1 < b.count && int(blockIdx.x) >= b.g0[s + 1]) ++s;
  rows_body<NG, RL>(b.scene[s], int(blockIdx.x) - b.g0[s], b.g0[s + 1] - b.g0[s]);
}

template <int NG>
__global__ __launch_bounds__(kBlock) void sgs_early_batch_kernel(IncBatch b) {
  int s = 0;
  while (s + 1 < b.count && int(blockIdx.x) >= b.g0[s + 1]) ++s;
  early_body<NG>(b.scene[s], int(blockIdx.x) - b.g0[s], b.g0[s + 1] - b.g0[s]);
}

// Scenes without a list phase (k_begin = k) leave at once.
template <int NG>
__global__ __launch_bounds__(kListBlock) void sgs_list_batch_kernel(IncBatch b) {
  int s = 0;
  while (s + 1 < b.count && int(blockIdx.x) >= b.g0[s + 1]) ++s;
  list_body<NG>(b.scene[s], int(blockIdx.x) - b.g0[s], b.g0[s + 1] - b.g0[s]);
}

// The rows form runs when the scene's best costs fit in LDS and a block has
// at most two columns per lane; otherwise the exchange form.
bool use_rows(int64_t n, int W) { return n <= kRowsMaxN && W <= kRowsMaxW; }

// A short greedy (few picks of a small scene) takes the exchange form's single
// launch whatever the schedule asked for: the rows form spends some 0.1 ms on
// its launches and first steps before its steps get cheaper than the exchange
// form's 5 to 7 us (k = 12 of 256 tokens: 115 against 160 us, 30 of 300: 210
// against 185, 51 of 1024: 390 against 292).  Same result.
// Blocks of a scene's greedy, and whether it is the rows form.  The rows form
// takes one block per kRowsPer tokens (up to one per compute unit: the early
// steps and the hits' row segments spread over more of the chip, 4096 tokens
// 0.05 ms faster than with one per 32), the exchange form one per 64.
constexpr int kRowsPer = 16;
constexpr int kShortN = 2048, kShortK = 20;
bool short_greedy(int64_t n, int64_t k) { return n <= kShortN && k <= kShortK; }
int inc_blocks(int64_t n, int cus, bool exchange, bool* rows) {
  const int nb = blocks_for(n, cus, kRowsPer);
  *rows = !exchange && use_rows(n, cols_for(n, nb));
  return *rows ? nb : blocks_for(n, cus, 64);
}

// The instance for the largest n and W of a launch.
constexpr int kRowsSmallN = kRowChunk * kWaves * 8;
const void* rows_kernel(int64_t n, int W) {
  if (n <= kRowsSmallN)
    return W <= 64 ? reinterpret_cast<const void*>(sgs_rows_kernel<1, 8>)
                   : reinterpret_cast<const void*>(sgs_rows_kernel<2, 8>);
  return reinterpret_cast<const void*>(sgs_rows_kernel<2, 16>);
}
const void* rows_batch_kernel(int64_t n, int W) {
  if (n <= kRowsSmallN)
    return W <= 64 ? reinterpret_cast<const void*>(sgs_rows_batch_kernel<1, 8>)
                   : reinterpret_cast<const void*>(sgs_rows_batch_kernel<2, 8>);
  return reinterpret_cast<const void*>(sgs_rows_batch_kernel<2, 16>);
}

// The step from which a scene's lists serve, and whether they do (there have
// to be some steps left to pay for building them: two launches of some 50 us).
// A step of the rows kernel takes 7 us, one of the list kernel 1.5; but lists built too early are long
// (n / 320: four scenes of 6272 tokens 4.0 ms instead of 2.6; n / 192: level).
// 12 steps: 20 picks of 1024 tokens 302 us with lists and 242 without, 28 of
// 2500 641 and 590, 61 of 6272 1283 and 1247.
int list_step(int64_t n) { return int(std::max<int64_t>(8, std::min<int64_t>(128, n / 128))); }
bool lists_for(int64_t n, int64_t k, int W) { return n <= kListMaxN && W <= kRowsMaxW && k > list_step(n) + 12; }

// Exchange slots and lists, the first pass's partial gains and scale, then
// (when the rows form may run) T.
constexpr int kPassParts = 3;   // row ranges of the first pass: 768 blocks at 16384 tokens, 192 at 4096
constexpr int kListOwnK = 128;  // up to this many picks the lists take the place of the rows of T
struct IncLayout {
  size_t part, scale, T, epart, epart_bytes, lists, ho_gain, ho_sel, ho_b, misc, total;
};
IncLayout inc_layout(int64_t n, int64_t k, bool compact) {
  IncLayout L;
  size_t o = layout(n, k).total;
  L.part = o; o += a256(size_t(kPassParts) * n * sizeof(long long));
  L.scale = o; o += 256;
  L.T = o;
  if (!compact && n <= kRowsMaxN) o += a256(size_t(n) * rows_ldt(n) * sizeof(float));
  // The early kernel's partial sums (rows schedule, n <= kEarlyMaxN): one
  // row per 64 tokens, and more in the lists' memory, which is free until the
  // lists are built.
  L.epart = o;
  L.epart_bytes = 0;
  const bool early = !compact && n <= kEarlyMaxN;
  if (early) o += a256(size_t(std::min<int64_t>(kMaxBlocks, (n + 63) / 64)) * early_ldp(n) * 8);
  // The candidate lists (n <= kListMaxN), and the hand-over between launches.
  L.lists = L.ho_gain = L.ho_sel = L.ho_b = L.misc = o;
  if (early) {
    L.lists = o;
    if (k > kListOwnK) o += a256(size_t(n) * kListCap * sizeof(uint2));
    L.epart_bytes = o - L.epart;
    L.ho_gain = o; o += a256(size_t(n) * 8);
    L.ho_sel = o;  o += a256(size_t(n));
    L.ho_b = o;    o += a256(size_t(rows_ldt(n)) * 4);
    L.misc = o;    o += a256(24 + 4 + size_t(kMaxBlocks) * 4);   // objective, exchanges, next step; the rest is spare
  }
  L.total = o;
  return L;
}
size_t inc_bytes(int64_t n, int64_t k, bool compact) { return inc_layout(n, k, compact).total; }

// nb: blocks; W64: the columns of one of a block per 64 tokens, whose gains compare
// exactly whatever the form's own split (a wider split is a group itself).
IncDev inc_dev(const SgsParams& p, char* w, int nb, int W64, bool rows) {
  const int W = cols_for(p.n, nb);
  const Layout L = layout(p.n, p.k);
  IncDev a{};
  a.C = p.cost;
  a.v = p.capacity;
  a.n = p.n;
  a.k = p.k;
  a.c0 = p.c0;
  a.selected = p.selected;
  a.step_gain = p.step_gain;
  a.step_obj = p.step_objective;
  a.assign = p.assign;
  a.list = reinterpret_cast<unsigned long long*>(w + L.list);
  a.lens = reinterpret_cast<unsigned long long*>(w + L.lens);
  a.cand = reinterpret_cast<unsigned long long*>(w + L.cand);
  a.abort = reinterpret_cast<unsigned int*>(w + L.ctrl);
  const WaitPolicy wp = wait_policy();
  a.poll_limit = wp.limit;
  a.abort_init = wp.preset;
  a.W = W;
  a.w_magic = w_magic_of(W);
  a.grp = std::max(W, W64);
  a.g_magic = w_magic_of(a.grp);
  const IncLayout M = inc_layout(p.n, p.k, !rows);
  a.T = rows ? reinterpret_cast<float*>(w + M.T) : nullptr;
  a.ldt = rows ? rows_ldt(p.n) : 0;
  a.part = reinterpret_cast<const long long*>(w + M.part);
  a.P = kPassParts;
  a.scale = reinterpret_cast<const int*>(w + M.scale);
  a.k_begin = 0;
  a.k_end = p.k;
  if (rows && p.n <= kEarlyMaxN) {
    a.ho_gain = reinterpret_cast<long long*>(w + M.ho_gain);
    a.ho_sel = reinterpret_cast<unsigned char*>(w + M.ho_sel);
    a.ho_b = reinterpret_cast<float*>(w + M.ho_b);
    a.ho_misc = reinterpret_cast<long long*>(w + M.misc);
  }
  if (rows && early_for(p.n, W)) {
    a.epart = reinterpret_cast<long long*>(w + M.epart);
    a.ldp = early_ldp(p.n);
    a.eshares = int(std::min<size_t>(nb, M.epart_bytes / (size_t(a.ldp) * 8)));
  }
  if (rows && lists_for(p.n, p.k, W)) {
    // Lists of their own, or (small budgets) at the start of the rows of T
    // that they replace.
    const bool own = p.k > kListOwnK;
    a.lists = own ? reinterpret_cast<uint2*>(w + M.lists) : reinterpret_cast<uint2*>(a.T);
    a.lcap = own ? kListCap : std::min(kListCap, a.ldt / 2);
    a.lstride = own ? size_t(kListCap) : size_t(a.ldt) / 2;
    a.lent = list_ent(p.n, W);
    a.llen = reinterpret_cast<unsigned int*>(w + L.list);   // and the best costs handed over (list_ho_b)
    a.k_end = list_step(p.n);
  }
  return a;
}

// The scale and the step-0 pass of one scene, ahead of the greedy's launch.
hipError_t launch_first_pass(const IncDev& a, hipStream_t stream) {
  inc_scale_kernel<<<1, kBlock, 0, stream>>>(a, const_cast<int*>(a.scale));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  long long* part = const_cast<long long*>(a.part);
  const dim3 grid((a.n + kPassCols - 1) / kPassCols, a.P);
  if (a.T && (a.abort_init & 2u))
    inc_first_pass_kernel<true, true><<<grid, kPassThreads, 0, stream>>>(a, part);
  else if (a.abort_init & 2u)
    inc_first_pass_kernel<false, true><<<grid, kPassThreads, 0, stream>>>(a, part);
  else if (a.T)
    inc_first_pass_kernel<true, false><<<grid, kPassThreads, 0, stream>>>(a, part);
  else
    inc_first_pass_kernel<false, false><<<grid, kPassThreads, 0, stream>>>(a, part);
  return hipGetLastError();
}

size_t lds_for(int W) { return size_t(W) * (8 + 4 + 4 + 1) + 16; }
size_t lds_rows(int W, int64_t n) { return size_t((W + 1) & ~1) * 8 + size_t(rows_ldt(n)) * 4 + size_t(W) + 16; }

hipError_t fits(const void* kernel, size_t lds, int threads = kBlock) {
  int per_cu = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, lds);
  if (e != hipSuccess) return e;
  return per_cu < 1 ? hipErrorCooperativeLaunchTooLarge : hipSuccess;
}

int device_cus(int* cus) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  return hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev);
}

// The instances for W columns a block.
const void* early_kernel(int W) {
  return W <= 64 ? reinterpret_cast<const void*>(sgs_early_kernel<1>) : reinterpret_cast<const void*>(sgs_early_kernel<2>);
}
const void* list_kernel(int W) {
  return W <= 64 ? reinterpret_cast<const void*>(sgs_list_kernel<1>) : reinterpret_cast<const void*>(sgs_list_kernel<2>);
}

// The greedy's launches; with `fused` the step-0 gains and T were written by
// fst_epilogue_sgs_kernel (and the scale before it), so the first pass is
// skipped and the gains come from its partial sums.
hipError_t run_incremental(const SgsParams& p, bool compact, const SgsFused* fused, hipStream_t stream,
                           SgsChecked* checked = nullptr) {
  int cus = 0;
  hipError_t e = hipError_t(device_cus(&cus));
  if (e != hipSuccess) return e;
  bool rows = false;
  const int nb = inc_blocks(p.n, cus, compact || (!checked && short_greedy(p.n, p.k)), &rows);
  const int W = cols_for(p.n, nb);
  // note_tie covers the exchange of the rows form with one column group.
  if (checked && (!rows || W > 64)) return hipSuccess;
  const void* kernel = rows ? rows_kernel(p.n, W) : reinterpret_cast<const void*>(sgs_inc_kernel);
  const size_t lds = rows ? lds_rows(W, p.n) : lds_for(W);
  if ((e = fits(kernel, lds)) != hipSuccess) return e;

  IncDev a = inc_dev(p, static_cast<char*>(p.workspace), nb, cols_for(p.n, blocks_for(p.n, cus, 64)), rows);
  if (fused) {
    a.part = fused->part;
    a.P = fused->P;
  }
  if (checked) {
    a.abort_init |= 2u;
    checked->unfit = a.abort + kUnfitWord;
    checked->tie = a.abort + kTieWord;
    checked->abort = a.abort;
    checked->scale = a.scale;
  }
  // The early kernel runs the first steps, while they improve many targets,
  // the rows kernel those up to the list phase (or the end), the list kernel
  // the rest.
  const bool early = a.epart != nullptr, lists = a.lists != nullptr;
  if (early && (e = fits(early_kernel(W), lds)) != hipSuccess) return e;
  if (lists && (e = fits(list_kernel(W), kListLds, kListBlock)) != hipSuccess) return e;
  sgs_inc_init_kernel<<<std::min(1024, (std::max(p.n, p.k) + 255) / 256), 256, 0, stream>>>(a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (!fused && (e = launch_first_pass(a, stream)) != hipSuccess) return e;
  if (early) {
    void* eargs[] = {&a};
    if ((e = hipLaunchCooperativeKernel(early_kernel(W), dim3(nb), dim3(kBlock), eargs, lds, stream)) != hipSuccess)
      return e;
    a.start = a.ho_misc + 2;
  }
  void* args[] = {&a};
  if ((e = hipLaunchCooperativeKernel(kernel, dim3(nb), dim3(kBlock), args, lds, stream)) != hipSuccess) return e;
  if (lists) {
    list_build_kernel<<<(p.n + 3) / 4, 256, 0, stream>>>(a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    a.k_begin = a.k_end;
    if ((e = hipLaunchCooperativeKernel(list_kernel(W), dim3(nb), dim3(kListBlock), args, kListLds, stream)) != hipSuccess)
      return e;
  }
  return launch_mark_aborted(a.abort, a.selected, a.k, stream);
}

}  // namespace

size_t sgs_inc_workspace_bytes(int64_t n, int64_t k, bool compact) { return inc_bytes(n, k, compact); }

hipError_t launch_sgs_incremental(const SgsParams& p, bool compact, hipStream_t stream) {
  return run_incremental(p, compact, nullptr, stream);
}

hipError_t launch_sgs_checked(const SgsParams& p, SgsChecked* checked, hipStream_t stream) {
  *checked = SgsChecked{};
  return run_incremental(p, false, nullptr, stream, checked);
}

// coverprune_prune: the rows schedule's workspace, then the epilogue's
// partial gains, [n / 64][n] 64-bit integers.
bool sgs_fused_fits(int64_t n) {
  int cus = 0;
  if (device_cus(&cus) != hipSuccess || n < 64 || n % 64 != 0) return false;
  return use_rows(n, cols_for(n, blocks_for(n, cus, kRowsPer)));
}

size_t sgs_fused_workspace_bytes(int64_t n, int64_t k) {
  return inc_bytes(n, k, false) + a256(size_t(n / 64) * size_t(n) * 8);
}

hipError_t sgs_fused_prepare(const SgsParams& p, SgsFused* f, hipStream_t stream) {
  int cus = 0;
  hipError_t e = hipError_t(device_cus(&cus));
  if (e != hipSuccess) return e;
  const int nb = blocks_for(p.n, cus, kRowsPer);
  IncDev a = inc_dev(p, static_cast<char*>(p.workspace), nb, cols_for(p.n, nb), true);
  f->T = a.T;
  f->ldt = a.ldt;
  f->part = reinterpret_cast<long long*>(static_cast<char*>(p.workspace) + inc_bytes(p.n, p.k, false));
  f->P = p.n / 64;
  f->scale = const_cast<int*>(a.scale);
  inc_scale_kernel<<<1, kBlock, 0, stream>>>(a, f->scale);
  return hipGetLastError();
}

hipError_t launch_sgs_fused(const SgsParams& p, const SgsFused& f, hipStream_t stream) {
  return run_incremental(p, false, &f, stream);
}

size_t sgs_inc_batch_workspace_bytes(const int64_t* n, const int64_t* k, int count, bool compact) {
  size_t total = 0;
  for (int s = 0; s < count; ++s) total += inc_bytes(n[s], k[s], compact);
  return total;
}

// One block per compute unit in all: every scene starts with one, then the
// scene with the most tokens per block gains one (up to its own cap of one
// block per `per` tokens, at most kMaxBlocks) until the units run out.
// Returns the blocks handed out.
static int share_blocks(const SgsParams* p, int count, int cus, int per, int* nb) {
  int used = count;
  for (int s = 0; s < count; ++s) nb[s] = 1;
  while (used < cus) {
    int best = -1, bw = 0;
    for (int s = 0; s < count; ++s)
      if (nb[s] < blocks_for(p[s].n, cus, per) && cols_for(p[s].n, nb[s]) > bw) {
        bw = cols_for(p[s].n, nb[s]);
        best = s;
      }
    if (best < 0) break;
    ++nb[best];
    ++used;
  }
  return used;
}

hipError_t launch_sgs_incremental_batch(const SgsParams* p, int count, bool compact, void* workspace,
                                        hipStream_t stream) {
  if (count < 1 || count > kMaxBatch) return hipErrorInvalidValue;
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
  if (count > cus) return hipErrorInvalidValue;
  bool rows = false;
  for (int s = 0; s < count; ++s) rows = rows || (!compact && !short_greedy(p[s].n, p[s].k));
  // Where some block has more than 64 columns the units ran out before any
  // scene reached its cap, so both shares are the same and every block is a
  // whole group, as the kernels for such blocks and the exchange form need.
  int nb[kMaxBatch], nb64[kMaxBatch];
  const int used = share_blocks(p, count, cus, rows ? kRowsPer : 64, nb);
  share_blocks(p, count, cus, 64, nb64);
  // The rows form when every scene allows it (one form per launch) and one is
  // not short, with the early and list kernels for the scenes they serve.
  // The list kernel serves when the scene with the most work (n k) has enough
  // steps left from its lists on to pay for two more launches, the scenes' builds, (beyond
  // kEarlyMinN) the early kernel, and, with more than 100 columns a block, pairs
  // that do not fit in LDS.  us without and with it: two scenes of 1000 tokens,
  // K = 50 373, 324; eight, K = 50 521, 540; four of 2000, K = 40 504, 548;
  // K = 60 608, 587; four of 6000, K = 100 1950, 1963; sixteen of 2000 (125
  // columns), K = 80 1311, 1412; eight of 4000, K = 80 1530, 1875.
  int big = 0;
  for (int s = 1; s < count; ++s)
    if (int64_t(p[s].n) * p[s].k > int64_t(p[big].n) * p[big].k) big = s;
  const int least = cols_for(p[big].n, nb[big]) > 100 ? 100 : p[big].n > kEarlyMinN ? 56 : 32 + 2 * count;
  bool early = false, lists = rows && p[big].k - list_step(p[big].n) > least;
  int wmax = 0, nmax = 0;
  for (int s = 0; s < count; ++s) {
    const int W = cols_for(p[s].n, nb[s]);
    rows = rows && use_rows(p[s].n, W);
    early = early || early_for(p[s].n, W);
    lists = lists && p[s].n <= kListMaxN && W <= kRowsMaxW;
    wmax = std::max(wmax, W);
    nmax = std::max(nmax, p[s].n);
  }
  lists = lists && rows;
  early = early && lists;
  IncBatch b{};
  b.count = count;
  b.g0[0] = 0;
  size_t lds = 0, off = 0;
  char* w = static_cast<char*>(workspace);
  for (int s = 0; s < count; ++s) {
    const int W = cols_for(p[s].n, nb[s]);
    IncDev& a = b.scene[s];
    a = inc_dev(p[s], w + off, nb[s], cols_for(p[s].n, nb64[s]), rows);
    if (!lists) {
      a.epart = nullptr;
      a.lists = nullptr;
      a.k_end = a.k;
    }
    b.g0[s + 1] = b.g0[s] + nb[s];
    lds = std::max(lds, rows ? lds_rows(W, p[s].n) : lds_for(W));
    off += inc_bytes(p[s].n, p[s].k, compact);
  }
  const bool one = wmax <= 64;   // one column group per block
  const void* kernel = rows ? rows_batch_kernel(nmax, wmax) : reinterpret_cast<const void*>(sgs_inc_batch_kernel);
  const void* ekernel = one ? reinterpret_cast<const void*>(sgs_early_batch_kernel<1>)
                            : reinterpret_cast<const void*>(sgs_early_batch_kernel<2>);
  const void* lkernel = one ? reinterpret_cast<const void*>(sgs_list_batch_kernel<1>)
                            : reinterpret_cast<const void*>(sgs_list_batch_kernel<2>);
  if ((e = fits(kernel, lds)) != hipSuccess) return e;
  if (early && (e = fits(ekernel, lds)) != hipSuccess) return e;
  if (lists && (e = fits(lkernel, kListLds, kListBlock)) != hipSuccess) return e;
  for (int s = 0; s < count; ++s) {
    sgs_inc_init_kernel<<<std::min(1024, (std::max(p[s].n, p[s].k) + 255) / 256), 256, 0, stream>>>(b.scene[s]);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = launch_first_pass(b.scene[s], stream)) != hipSuccess) return e;
  }
  void* args[] = {&b};
  if (early) {
    if ((e = hipLaunchCooperativeKernel(ekernel, dim3(used), dim3(kBlock), args, lds, stream)) != hipSuccess) return e;
    for (int s = 0; s < count; ++s)
      if (b.scene[s].epart) b.scene[s].start = b.scene[s].ho_misc + 2;
  }
  if ((e = hipLaunchCooperativeKernel(kernel, dim3(used), dim3(kBlock), args, lds, stream)) != hipSuccess) return e;
  bool any = false;
  for (int s = 0; s < count; ++s) any = any || b.scene[s].lists;
  if (any) {
    for (int s = 0; s < count; ++s) {
      IncDev& a = b.scene[s];
      a.k_begin = a.k_end;
      if (!a.lists) continue;
      list_build_kernel<<<(p[s].n + 3) / 4, 256, 0, stream>>>(a);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if ((e = hipLaunchCooperativeKernel(lkernel, dim3(used), dim3(kListBlock), args, kListLds, stream)) != hipSuccess)
      return e;
  }
  for (int s = 0; s < count; ++s)
    if ((e = launch_mark_aborted(b.scene[s].abort, b.scene[s].selected, b.scene[s].k, stream)) != hipSuccess) return e;
  return hipSuccess;
}

}  // namespace cp
