// Shared parts of the persistent greedy kernels that keep their gains in
// exact fixed point: the incremental form (k_sgs_inc.hip) and the local form
// (k_sgs_local.hip), Sec. 3.5.  Both run one cooperative launch of one block
// per compute unit; block b owns tokens [b W, (b + 1) W).
//
// The exchanges are per-block slots rather than counters: a slot holds the
// value together with the step it belongs to, every block reads all slots in
// parallel (one thread per slot), and no address takes more than one writer,
// so a step costs two round trips through memory instead of two grid
// barriers of serialized atomic increments.  Slots, lists and lengths are
// written and read with device-scope atomic operations, coherent across the
// chip's L2 caches without fences; a block's list writes are complete at the
// workgroup barrier before its thread 0 publishes the length.  A slot is only
// rewritten after every block has read it: a block can publish step l + 1's
// values only after reading every block's step-l + 1 candidate, which each
// block publishes only after it has consumed step l.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>

#include "common.h"
#include "fixed_point.h"
#include "launch.h"

namespace cp {
namespace {

constexpr int kBlock = 512;
constexpr int kWaves = kBlock / 64;
constexpr int kMaxBlocks = 256;    // at most one block per compute unit
// Exchange slots sit one per 128-byte line: packed 8 bytes apart, 16 blocks
// on different XCDs would write into the line that every block is polling.
constexpr int kSlotStride = 16;
constexpr int kIndexBits = 20;     // candidate: [epoch | 43-bit gain | 20-bit inverted index]
constexpr unsigned long long kIndexMask = (1ull << kIndexBits) - 1ull;
constexpr unsigned long long kEpoch = 1ull << 63;
constexpr unsigned long long kNoCandidate = 1ull;   // below every real candidate
// The list kernel's words hold exact gains (62 bits); bit 62 marks "none".
constexpr unsigned long long kNoGain = 1ull << 62;
constexpr int kListWord = 8;                        // first of a slot's words that the list kernel uses
// Every wait in the kernel is bounded (give_up in common.h): a wait that
// gives up raises the abort flag, every block leaves its waits and returns,
// and a kernel after the launch fills selected[] with -1.

struct IncDev {
  const float* C;
  const float* v;
  int n, k;
  float c0;
  int32_t* selected;
  double* step_gain;
  double* step_obj;
  int32_t* assign;
  unsigned long long* list;   // [blocks][W][2]: (row | v << 32), (old b | new b << 32)
  unsigned long long* lens;   // [blocks] (step + 1) << 32 | slice length
  unsigned long long* cand;   // [2][blocks] packed candidate | epoch << 63
  unsigned int* abort;        // set when a wait gives up
  unsigned int poll_limit;    // polls before a wait gives up (WaitPolicy)
  unsigned int abort_init;    // bit 0: the abort flag's value at launch (WaitPolicy); bit 1: check the data
  int W;                      // rows and columns per block
  unsigned int w_magic;       // floor(2^32 / W) + 1: block_of(c) = c / W by one high multiply
  float* T;                   // rows form only: [n][ldt] source-major copy, T[s][t] = C(s, t)
  int ldt;                    // its row stride, n rounded up to a whole 256-row chunk
  unsigned int g_magic;       // floor(2^32 / grp) + 1: group_of(c) = c / grp
  const long long* part;      // incremental form: [P][n] step-0 gains summed over P row ranges
  int P;
  int grp;                    // consecutive columns whose gains compare exactly (pack_key); at least W
  const int* scale;           // incremental form: the fixed-point exponent S
  // Rows schedule in several launches with a hand-over (see k_sgs_inc.hip):
  // the steps of this launch and the state handed from one to the next.
  int k_begin, k_end;         // steps [k_begin, k_end); [0, k) for a single launch
  long long* ho_gain;         // [n] running gains
  unsigned char* ho_sel;      // [n] chosen flags
  float* ho_b;                // [ldt] best costs
  long long* ho_misc;         // [0] objective in fixed point, [1] exchanges so far, [2] next step
  uint2* lists;               // candidate c's list at lists + c lstride: (target, cost) pairs
  size_t lstride;
  int lcap;                   // pairs a list holds; a candidate with more keeps its row of T
  int lent;                   // pairs of its own candidates that a block holds
  unsigned int* llen;         // [n] pairs of each candidate
  // Early steps of the rows schedule (sgs_early_kernel): each block's partial
  // gain changes of every column, and the step a launch after it starts from
  // (null: k_begin).
  long long* epart;           // [eshares][ldp]: columns 0 .. n - 1, then the objective's change
  int ldp, eshares;
  const long long* start;
};

// With the data checked, word kUnfitWord after the abort flag is set when they
// are outside the fixed point's domain, and the launches after the first pass
// leave at once.
constexpr int kUnfitWord = 16;
__device__ __forceinline__ bool unfit(const IncDev& a) { return (a.abort_init & 2u) && a.abort[kUnfitWord]; }

// Also with the data checked: word kTieWord is set when an exact gain, not
// its key, had to decide between candidates (the kernels in flight go on).
constexpr int kTieWord = 17;
__device__ __forceinline__ void note_tie(const IncDev& a) {
  if (a.abort_init & 2u) atomicOr(a.abort + kTieWord, 1u);
}

// The block that owns column c: c / W as the high word of c times
// floor(2^32 / W) + 1, exact for c < 2^18 and 2 <= W <= 2^13 (the product
// exceeds 2^32 c / W by less than c, which moves c / W by less than 2^-14,
// below the gap 1 / W to the next integer).  W = 1 only with n = 1 (a
// grid has one block per 16 tokens at most), where the multiplier wraps to
// 0 and column 0's block is 0.
__device__ __forceinline__ int block_of(const IncDev& a, int c) { return int(__umulhi(unsigned(c), a.w_magic)); }
inline unsigned int w_magic_of(int W) { return unsigned(0xffffffffu / unsigned(W)) + 1u; }
__device__ __forceinline__ int group_of(const IncDev& a, int c) { return int(__umulhi(unsigned(c), a.g_magic)); }

struct Layout {
  size_t list, lens, cand, ctrl, total;
};

size_t a256(size_t x) { return (x + 255) / 256 * 256; }

// One block per `per` tokens, at most one per compute unit.
int blocks_for(int64_t n, int cus, int per) {
  return int(std::max<int64_t>(1, std::min<int64_t>(std::min(cus, kMaxBlocks), (n + per - 1) / per)));
}

// Columns a block of nb.
int cols_for(int64_t n, int nb) { return int((n + nb - 1) / nb); }

// Sized for the largest grid (kMaxBlocks blocks of W = ceil(n / blocks) rows).
Layout layout(int64_t n, int64_t k) {
  (void)k;
  Layout L;
  size_t o = 0;
  L.list = o; o += a256(size_t(n + kMaxBlocks) * 16);
  L.lens = o; o += a256(size_t(kMaxBlocks) * kSlotStride * 8);
  L.cand = o; o += a256(size_t(2 * kMaxBlocks) * kSlotStride * 8);
  L.ctrl = o; o += 256;
  L.total = o;
  return L;
}

// Block b's candidate slot of slot set `set` (set = step % 2), and its
// slice-length slot.
__host__ __device__ __forceinline__ unsigned long long* cand_slot(unsigned long long* cand, int set, int b) {
  return cand + (size_t(set) * kMaxBlocks + b) * kSlotStride;
}
__host__ __device__ __forceinline__ unsigned long long* lens_slot(unsigned long long* lens, int b) {
  return lens + size_t(b) * kSlotStride;
}

// The order of candidates.  A key holds the nonnegative gain truncated to its
// top 43 bits (relative resolution 2^-31), then the inverted index: larger
// gain first, then smaller index.  Candidates of one group (grp consecutive
// columns) compare by their exact gains, then by index; as a group's columns
// are consecutive, the order over all is: larger truncated gain, lower group,
// larger exact gain, smaller index.  It does not depend on how the columns are
// split over the blocks.  Indices are below 2^18, so every real candidate
// exceeds kNoCandidate.
__device__ __forceinline__ unsigned long long pack_key(double g, int idx) {
  const unsigned long long gb = (unsigned long long)__double_as_longlong(g) >> (kIndexBits + 1);
  return (gb << kIndexBits) | (kIndexMask - (unsigned long long)idx);
}

// The key's order for an exact gain (-1: none, below all): the top 43 bits
// of its float64 value, which scaling by 2^-S does not change, plus one.
__device__ __forceinline__ unsigned long long gain_key(long long g) {
  return g < 0 ? 0ull : ((unsigned long long)__double_as_longlong(double(g)) >> (kIndexBits + 1)) + 1ull;
}
__device__ __forceinline__ unsigned long long gain_word(long long g) { return g < 0 ? kNoGain : (unsigned long long)g; }
__device__ __forceinline__ long long word_gain(unsigned long long x) {
  return (x & kNoGain) ? -1ll : (long long)(x & ~kEpoch);
}

// Epoch bit of the candidates of exchange l (the step, unless steps skip
// their exchange), kept in slot set l % 2: it flips between consecutive uses
// of a set and is never the zero of a fresh workspace for exchanges 0 and 1.
__device__ __forceinline__ unsigned long long epoch_of(int step) {
  return ((step >> 1) & 1) ? 0ull : kEpoch;
}

__global__ void sgs_inc_init_kernel(IncDev a) {
  const int gt = blockIdx.x * blockDim.x + threadIdx.x, nt = gridDim.x * blockDim.x;
  for (int s = gt; s < kMaxBlocks; s += nt) a.lens[size_t(s) * kSlotStride] = 0ull;
  for (int i = gt; i < 2 * kMaxBlocks * kSlotStride; i += nt) a.cand[i] = 0ull;
  for (int j = gt; j < a.n; j += nt)
    if (a.assign) a.assign[j] = -1;
  if (gt == 0) *a.abort = a.abort_init & 1u;
  if (gt == 0) a.abort[kUnfitWord] = a.abort[kTieWord] = 0u;
}

// Wave reductions without LDS traffic: DPP moves within each row of 16
// lanes, in the pattern swap neighbours, swap pairs, mirror halves of 8,
// mirror the row (after each step every lane of a group of 2, 4, 8, 16 holds
// the group's result), then the four row results read from lanes 0, 16, 32
// and 48.  Every lane of the wave must be active.
constexpr int kDppSteps[4] = {0xB1, 0x4E, 0x141, 0x140};   // quad_perm [1,0,3,2], [2,3,0,1], row_half_mirror, row_mirror

__device__ __forceinline__ unsigned long long lane_u64(unsigned long long x, int r) {
  return ((unsigned long long)__builtin_amdgcn_readlane(unsigned(x >> 32), r) << 32) |
         unsigned(__builtin_amdgcn_readlane(unsigned(x), r));
}


__device__ __forceinline__ unsigned wave_max_u32(unsigned x) {
  x = max(x, unsigned(__builtin_amdgcn_mov_dpp(int(x), kDppSteps[0], 0xf, 0xf, false)));
  x = max(x, unsigned(__builtin_amdgcn_mov_dpp(int(x), kDppSteps[1], 0xf, 0xf, false)));
  x = max(x, unsigned(__builtin_amdgcn_mov_dpp(int(x), kDppSteps[2], 0xf, 0xf, false)));
  x = max(x, unsigned(__builtin_amdgcn_mov_dpp(int(x), kDppSteps[3], 0xf, 0xf, false)));
  return max(max(unsigned(__builtin_amdgcn_readlane(int(x), 0)), unsigned(__builtin_amdgcn_readlane(int(x), 16))),
             max(unsigned(__builtin_amdgcn_readlane(int(x), 32)), unsigned(__builtin_amdgcn_readlane(int(x), 48))));
}

// The maximum over lanes 0 .. 31, in every lane.
__device__ __forceinline__ unsigned half_max_u32(unsigned x) {
  x = max(x, unsigned(__builtin_amdgcn_mov_dpp(int(x), kDppSteps[0], 0xf, 0xf, false)));
  x = max(x, unsigned(__builtin_amdgcn_mov_dpp(int(x), kDppSteps[1], 0xf, 0xf, false)));
  x = max(x, unsigned(__builtin_amdgcn_mov_dpp(int(x), kDppSteps[2], 0xf, 0xf, false)));
  x = max(x, unsigned(__builtin_amdgcn_mov_dpp(int(x), kDppSteps[3], 0xf, 0xf, false)));
  return max(unsigned(__builtin_amdgcn_readlane(int(x), 0)), unsigned(__builtin_amdgcn_readlane(int(x), 16)));
}

__device__ __forceinline__ int wave_sum_i32(int x) {
  x += __builtin_amdgcn_mov_dpp(x, kDppSteps[0], 0xf, 0xf, false);
  x += __builtin_amdgcn_mov_dpp(x, kDppSteps[1], 0xf, 0xf, false);
  x += __builtin_amdgcn_mov_dpp(x, kDppSteps[2], 0xf, 0xf, false);
  x += __builtin_amdgcn_mov_dpp(x, kDppSteps[3], 0xf, 0xf, false);
  return __builtin_amdgcn_readlane(x, 0) + __builtin_amdgcn_readlane(x, 16) + __builtin_amdgcn_readlane(x, 32) +
         __builtin_amdgcn_readlane(x, 48);
}

// A workgroup barrier that orders LDS only: outstanding global loads stay in
// flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The 64-bit maximum as 32-bit ones: the largest high word, then the low
// word of the one lane that holds it, or, when several do, the largest of
// their low words (32-bit steps take one compare-select where a 64-bit step
// takes three).
__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long x) {
  const unsigned hi = unsigned(x >> 32);
  const unsigned hm = wave_max_u32(hi);
  const unsigned long long tie = __ballot(hi == hm);
  unsigned lm;
  if (__popcll(tie) == 1)
    lm = unsigned(__builtin_amdgcn_readlane(int(unsigned(x)), __builtin_ctzll(tie)));
  else
    lm = wave_max_u32(hi == hm ? unsigned(x) : 0u);
  return ((unsigned long long)hm << 32) | lm;
}

__device__ __forceinline__ long long wave_sum_i64(long long x) {
  x += (long long)dpp_u64<kDppSteps[0]>((unsigned long long)x);
  x += (long long)dpp_u64<kDppSteps[1]>((unsigned long long)x);
  x += (long long)dpp_u64<kDppSteps[2]>((unsigned long long)x);
  x += (long long)dpp_u64<kDppSteps[3]>((unsigned long long)x);
  return (long long)(lane_u64((unsigned long long)x, 0) + lane_u64((unsigned long long)x, 16) +
                     lane_u64((unsigned long long)x, 32) + lane_u64((unsigned long long)x, 48));
}

__device__ __forceinline__ int wave_min_i32(int x) {
  int y;
  y = __builtin_amdgcn_mov_dpp(x, kDppSteps[0], 0xf, 0xf, false); x = y < x ? y : x;
  y = __builtin_amdgcn_mov_dpp(x, kDppSteps[1], 0xf, 0xf, false); x = y < x ? y : x;
  y = __builtin_amdgcn_mov_dpp(x, kDppSteps[2], 0xf, 0xf, false); x = y < x ? y : x;
  y = __builtin_amdgcn_mov_dpp(x, kDppSteps[3], 0xf, 0xf, false); x = y < x ? y : x;
  int m = __builtin_amdgcn_readlane(x, 0);
#pragma unroll
  for (int r = 16; r < 64; r += 16) {
    y = __builtin_amdgcn_readlane(x, r);
    m = y < m ? y : m;
  }
  return m;
}

// Inclusive prefix sum over the lanes of a wave (every lane active).
__device__ __forceinline__ int wave_scan_incl(int x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  return x;
}

// Sum over the block of 64-bit integers, result in every thread.
__device__ long long block_sum_i64(long long x, long long* sg) {
  x = wave_sum_i64(x);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sg[w] = x;
  __syncthreads();
  long long s = 0;
#pragma unroll
  for (int q = 0; q < kWaves; ++q) s += sg[q];
  __syncthreads();
  return s;
}

// Poll *p until pred(value) holds; false if the launch is aborting (this
// wait gave up, or another one did).
template <class Pred>
__device__ bool wait_slot(const unsigned long long* p, unsigned int* abort, unsigned int limit, Pred pred,
                          unsigned long long& x) {
  for (unsigned int spins = 0;; ++spins) {
    x = get(p);
    if (pred(x)) return true;
    if (give_up(spins, limit, abort)) return false;
    __builtin_amdgcn_s_sleep(1);
  }
}

// Inclusive prefix sum over the block (thread order), result in every thread.
__device__ int block_inclusive_scan(int x, int* swt) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) swt[w] = x;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kWaves; ++q)
    if (q < w) x += swt[q];
  __syncthreads();
  return x;
}

// Fixed-order block sum, result in every thread.
__device__ double block_sum_all(double x, double* sd) {
  x = wave_sum(x);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sd[w] = x;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < kWaves; ++q) s += sd[q];
  __syncthreads();
  return s;
}

// Thread t's part of sum_j fx(v_j c0, S), the objective at b = c0 (exact
// integers, so the parts and their total do not depend on the order): j = t,
// t + kBlock, ..., eight loads in flight at a time (a load whose result the
// next iteration needs waits for itself otherwise).
__device__ __forceinline__ long long fx_capacity_part(const float* v, int n, float c0, int S) {
  long long x = 0;
  constexpr int U = 8;
  for (int j0 = threadIdx.x; j0 < n; j0 += kBlock * U) {
    float vv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) vv[u] = v[min(j0 + u * kBlock, n - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j0 + u * kBlock < n) x += fx(double(vv[u]) * double(c0), S);
  }
  return x;
}

// Block maximum, result in every thread.
__device__ double block_max_all(double x, double* sd) {
  x = wave_max(x);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sd[w] = x;
  __syncthreads();
  double s = sd[0];
#pragma unroll
  for (int q = 1; q < kWaves; ++q) s = fmax(s, sd[q]);
  __syncthreads();
  return s;
}

// Of the lanes in `tie` (not empty), whose candidates' truncated gains are
// equal, the one whose candidate (of a group, with a gain and an index) comes
// first.  Every lane of the wave is active.
__device__ __forceinline__ int first_of(unsigned long long tie, int group, long long g, int idx) {
  if (__popcll(tie) > 1) {
    bool in = (tie >> (threadIdx.x & 63)) & 1ull;
    const int gm = wave_min_i32(in ? group : INT_MAX);
    in = in && group == gm;
    const unsigned long long top = wave_max_u64(in ? (unsigned long long)(g + 1) : 0ull);
    in = in && (unsigned long long)(g + 1) == top;
    const int im = wave_min_i32(in ? idx : INT_MAX);
    tie = __ballot(in && idx == im);
  }
  return __builtin_ctzll(tie);
}

// The block's first unchosen column in the order of candidates, published as
// its candidate for the step.  With at most 64 columns wave 0 does it alone,
// one column per lane, and no barrier follows: the callers' next step begins
// with one (read_winner), and the gains and chosen flags it reads were last
// written by wave 0 itself.  A block is one group here, so the exact gains
// decide.
__device__ __forceinline__ unsigned long long column_key(const long long* sG, const unsigned char* ssel, int lo, int i,
                                                         int cnt, int S) {
  return i < cnt && !ssel[i] ? pack_key(fx_to_double(sG[i], S), lo + i) : kNoCandidate;
}
// The first of one wave's columns (one a lane): its lane and key (top: the
// largest key, whose truncated gain others may share), and the best key of
// the others.
struct WaveBest {
  unsigned long long key, second;
  int lane;
};
__device__ __forceinline__ WaveBest wave_best(const IncDev& a, const long long* sG, unsigned long long mine, int lo) {
  const int lane = threadIdx.x & 63;
  WaveBest r;
  r.key = wave_max_u64(mine);
  r.lane = (int(kIndexMask - (r.key & kIndexMask)) - lo) & 63;
  r.second = wave_max_u64(mine == r.key ? kNoCandidate : mine);
  if (r.second > kNoCandidate && (r.second >> kIndexBits) == (r.key >> kIndexBits)) {
    const unsigned long long tie = __ballot(mine > kNoCandidate && (mine >> kIndexBits) == (r.key >> kIndexBits));
    const long long g = (tie >> lane) & 1ull ? sG[lane] : 0;
    r.lane = first_of(tie, group_of(a, lo + lane), g, lo + lane);
    if (((tie >> lane) & 1ull) && g != sG[r.lane]) note_tie(a);
    r.key = lane_u64(mine, r.lane);
    r.second = wave_max_u64(lane == r.lane ? kNoCandidate : mine);
  }
  return r;
}
__device__ __forceinline__ void publish_argmax(const long long* sG, const unsigned char* ssel, int lo,
                                               int cnt, int S, unsigned long long* slot, unsigned long long epoch,
                                               unsigned long long* su) {
  if (cnt <= 64) {
    if (threadIdx.x >= 64) return;
    const int i = threadIdx.x;
    const unsigned long long g1 = i < cnt && !ssel[i] ? (unsigned long long)sG[i] + 1ull : 0ull;   // 0: no candidate
    const unsigned long long top = wave_max_u64(g1);
    const int first = __builtin_ctzll(__ballot(g1 == top));
    if (i == 0) put(slot, (top ? pack_key(fx_to_double((long long)(top - 1), S), lo + first) : kNoCandidate) | epoch);
    return;
  }
  __shared__ int si[kWaves];
  long long g = -1;
  int gi = INT_MAX;
  for (int i = threadIdx.x; i < cnt; i += kBlock)
    if (!ssel[i] && sG[i] > g) {   // increasing i: ties keep the smaller index
      g = sG[i];
      gi = lo + i;
    }
  unsigned long long top = wave_max_u64((unsigned long long)(g + 1));   // 0: no candidate
  gi = wave_min_i32((unsigned long long)(g + 1) == top ? gi : INT_MAX);
  if ((threadIdx.x & 63) == 0) {
    su[threadIdx.x >> 6] = top;
    si[threadIdx.x >> 6] = gi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < kWaves; ++q)
      if (su[q] > top || (su[q] == top && si[q] < gi)) {
        top = su[q];
        gi = si[q];
      }
    put(slot, (top ? pack_key(fx_to_double((long long)(top - 1), S), gi) : kNoCandidate) | epoch);
  }
  __syncthreads();
}

// The step's winner: thread i < nb waits for block i's candidate of this
// epoch; the largest wins (the same in every block).  Returns -1 when the
// launch is aborting.
__device__ int read_winner(const unsigned long long* slots, unsigned long long epoch, int nb,
                           unsigned int* abort, unsigned int limit, unsigned long long* su, int* sflag) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  unsigned long long best = 0ull;
  if (tid == 0) *sflag = 0;
  __syncthreads();
  if (tid < nb) {
    unsigned long long x;
    if (wait_slot(slots + size_t(tid) * kSlotStride, abort, limit,
                  [epoch](unsigned long long v) { return (v & kEpoch) == epoch; }, x))
      best = x & ~kEpoch;
    else
      *sflag = 1;
  }
  best = wave_max_u64(best);
  if (lane == 0) su[w] = best;
  __syncthreads();
  unsigned long long m = su[0];
#pragma unroll
  for (int q = 1; q < kWaves; ++q) m = su[q] > m ? su[q] : m;
  const bool aborting = *sflag != 0;
  __syncthreads();
  return aborting ? -1 : int(kIndexMask - (m & kIndexMask));
}

// The form of publish_argmax and read_winner for kernels that predict
// the next winner (at most 64 columns a block): the block's best key in word 0
// of its slot, its second-best in word 1 and, where a group can reach over
// several blocks (SPANS), the best one's exact gain in word 2, each with the
// epoch bit.
template <bool SPANS>
__device__ __forceinline__ void publish_rows(const IncDev& a, const long long* sG, const unsigned char* ssel, int lo,
                                             int cnt, int S, unsigned long long* slot, unsigned long long epoch) {
  if (threadIdx.x >= 64) return;
  if (!SPANS) {
    // The block is a group: its first column by exact gain, as in publish_argmax.
    const int i = threadIdx.x;
    const unsigned long long g1 = i < cnt && !ssel[i] ? (unsigned long long)sG[i] + 1ull : 0ull;
    const unsigned long long key = g1 ? pack_key(fx_to_double((long long)(g1 - 1), S), lo + i) : kNoCandidate;
    const int first = __builtin_ctzll(__ballot(g1 == wave_max_u64(g1)));
    const unsigned long long second = wave_max_u64(i == first ? kNoCandidate : key);
    if (i < 2) put(slot + i, (i ? second : lane_u64(key, first)) | epoch);
    return;
  }
  const WaveBest best = wave_best(a, sG, column_key(sG, ssel, lo, threadIdx.x, cnt, S), lo);
  unsigned long long word = threadIdx.x ? best.second : best.key;
  // One store of three lanes; without a candidate the gain is not read.
  const unsigned long long g = lane_u64((unsigned long long)sG[int(threadIdx.x) < cnt ? threadIdx.x : 0], best.lane);
  if (threadIdx.x == 2) word = g & ~kEpoch;
  if (threadIdx.x < 3) put(slot + threadIdx.x, word | epoch);
}

// Of the blocks' best candidates with the truncated gain of m (the one with
// the smallest index, so the lowest group), the first one's index, the same in
// every wave.
__device__ __forceinline__ int first_of_blocks(const IncDev& a, unsigned long long m, int nb,
                                            const unsigned long long* sk1, const unsigned long long* sk3) {
  const int lane = threadIdx.x & 63;
  const int gm = group_of(a, int(kIndexMask - (m & kIndexMask)));
  unsigned long long best = 0ull;
  int bi = INT_MAX;
#pragma unroll 1
  for (int b = lane; b < nb; b += 64) {             // increasing b: ties keep the smaller index
    const int i = int(kIndexMask - (sk1[b] & kIndexMask));
    if (sk1[b] > kNoCandidate && (sk1[b] >> kIndexBits) == (m >> kIndexBits) && group_of(a, i) == gm && sk3[b] + 1 > best) {
      best = sk3[b] + 1;
      bi = i;
    }
  }
  const unsigned long long top = wave_max_u64(best);
  return wave_min_i32(best == top ? bi : INT_MAX);
}

// read_winner for such slots: thread i < nb polls words 0 and 1 of block i's
// slot and stores them (epoch bits cleared) in sk1 and sk2.  Returns the
// winner's index, -1 when the launch is aborting.  With SPANS the blocks whose
// truncated gain is the winner's are told apart by word 2 (sk3), read only
// then; sflag has a second word for that.
template <bool SPANS>
__device__ int read_winner_rows(const IncDev& a, const unsigned long long* slots, unsigned long long epoch, int nb,
                                unsigned long long* su, int* sflag, unsigned long long* sk1, unsigned long long* sk2,
                                unsigned long long* sk3) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  unsigned long long own = 0ull;
  if (tid == 0) {
    sflag[0] = 0;
    if (SPANS) sflag[1] = 0;
  }
  __syncthreads();
  if (tid < nb) {
    const unsigned long long* p = slots + size_t(tid) * kSlotStride;
    bool done = false;
    for (unsigned int spins = 0; !done; ++spins) {
      const unsigned long long x0 = get(p), x1 = get(p + 1);
      if ((x0 & kEpoch) == epoch && (x1 & kEpoch) == epoch) {
        own = x0 & ~kEpoch;
        sk1[tid] = own;
        sk2[tid] = x1 & ~kEpoch;
        done = true;
      } else {
        if (give_up(spins, a.poll_limit, a.abort)) {
          sflag[0] = 1;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
  }
  const unsigned long long best = wave_max_u64(own);
  if (lane == 0) su[w] = best;
  __syncthreads();
  unsigned long long m = su[0];
#pragma unroll
  for (int q = 1; q < kWaves; ++q) m = su[q] > m ? su[q] : m;
  const bool tied = own > kNoCandidate && (own >> kIndexBits) == (m >> kIndexBits);
  if (SPANS && tied && own != m) sflag[1] = 1;
  const bool aborting = sflag[0] != 0;
  __syncthreads();
  if (aborting) return -1;
  if (SPANS && sflag[1]) {
    if (tied) {
      unsigned long long x = 0ull;
      if (!wait_slot(slots + size_t(tid) * kSlotStride + 2, a.abort, a.poll_limit,
                     [epoch](unsigned long long v) { return (v & kEpoch) == epoch; }, x))
        sflag[0] = 1;
      sk3[tid] = x & ~kEpoch;
    }
    __syncthreads();
    if (sflag[0]) return -1;
    if (tied && sk3[tid] != sk3[block_of(a, int(kIndexMask - (m & kIndexMask)))]) note_tie(a);
    return first_of_blocks(a, m, nb, sk1, sk3);
  }
  return int(kIndexMask - (m & kIndexMask));
}

}  // namespace
}  // namespace cp
