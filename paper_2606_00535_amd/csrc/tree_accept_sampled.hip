// Sampled tree acceptance at temperature tau: speculative sampling's accept-or-resample rule (the paper's
// Section 1 and Section 2, "Speculative decoding"; its Table 2 runs at temperature 1) applied down the tree.
//
// The rule.  p and q are the target's and the draft's softmax(logits / tau) at a node.  Its children are tested
// in index order: child c, carrying token x, is kept with probability min(1, r(x) / q(x)), and the walk descends
// into the first kept child; after a rejection r becomes max(r - q, 0) renormalised (unchanged if that is zero).
// r starts as p.  Where no child is kept (or at a leaf) the emitted token is drawn from r.  Child c is decided
// by the caller's uniform u[c]; the emitted token by u[0], through the inverse CDF of r.
//
// The residual after k rejections at a node has the closed form r_k = max(p - C_k q, 0) / D_k, with C_0 = 0,
// D_0 = 1, and after rejecting one more child C_{k+1} = C_k + D_k, D_{k+1} = sum_x max(p - C_{k+1} q, 0) (both
// unchanged when that sum is zero).  So the children of a node need only the node's own p and q.  A vocabulary
// row is cut into pieces, a workgroup each, which keep their entries in registers and
//   (1) compute the piece's maxima and sums of exp((l - max) / tau), target and draft, exchange them, and merge
//       the row's statistics themselves, in the same order (the same bits everywhere): p and q;
//   (2) take the node's children in index order: child c, token x, is decided by the piece holding x
//       (u q(x) D < max(p(x) - C q(x), 0)) against the state its earlier siblings left; the pieces exchange that
//       decision with their parts of c's residual mass sum max(p - (C + D) q, 0), which moves the state;
//   (3) draw the token emitted if the walk ends at the node: the prefix of the piece masses (of the last child
//       that moved the state, or of p) names the piece where the cumulative mass first exceeds u0 * total, and
//       that piece finds the token by a block scan.
// Three forms place this work.  Only the rows that the walk visits matter -- the root's and each kept child's --
// but which they are is known only as the walk goes:
//   * walk form: a workgroup per piece of every sequence.  The sequence's pieces take the walk's rows one after
//     the other, deciding alike; only those rows are read.  Time grows with the walk's length.
//     16 trees of 128 nodes x 152064 entries: 112 us, against 1.76 ms for every row's pieces in parallel (there
//     the fp64 exponentials of 2048 rows bound the call; here the exponentials and loads of the visited rows,
//     about 10 us a row, and the exchanges, about 1.7 us each).
//   * row form: a workgroup per piece of every row of the tree, all at once; the sequence's last row to finish
//     walks the decisions by ballots.  Time grows with the number of rows, not with the walk's length.  60 nodes x
//     32000 entries: 24.5 us (28.6 with the statistics merged through a counter and a second round of loads, and
//     butterfly reductions through LDS); a chain of exchanges as long as the widest node's children.
//   * either form: a sequence whose tree has no path of more than `max_visits` nodes is walked; any other takes its
//     rows all the same, in turn by a few clusters, so that a long path that is kept costs no more than that.  Both
//     kinds of workgroup are launched and read the paths off the parents, and one kind leaves at once.
// Probabilities are fp64, so that the integer outcome is decided in the precision of the definition; exp is
// Tang's table-driven method.
//
// Exchange.  The pieces of a row (row form), of several rows (either form) or of a sequence (walk form) are a
// cluster.  In step s = 1, 2, ... (a row's statistics, and in the walk form every child tested) every piece stores its
// few words, each 48 bits of data beside the step's number, to its own slot, and one wave polls all slots of the
// cluster, lane k the slot of piece k, until every word carries the step's number: one store and one load of latency,
// with no counter in between.  Slots alternate between two places: a piece
// writes step s + 2 only after it has read every piece's step s + 1, which each wrote after reading step s.
// A slot holds anything at entry; each piece clears its own and counts itself in on the cluster's counter, and
// nobody reads a slot before that count is whole (the pieces that left are counted apart, so that it means what it
// says also where others gave up and left early).  (A row of one piece has nothing to exchange.)  The row form
// has slots for the statistics only: a child's residual mass is summed over the pieces by one atomic each, in
// fixed point (units of 2^-51, so the sum does not depend on the order of arrival), with the arrivals above it
// and the decision between them, and the pieces poll that word.
//
// Forward progress.  A piece waits only for the other pieces of its own cluster, which are consecutive
// workgroups and wait for nothing outside it.  Workgroups are dispatched in blockIdx order and at most 64 make a
// cluster, so every wait ends.  Waits are nevertheless bounded (0.2 s by default), after which the results are
// unspecified and the workspace's failure flag is set: a piece whose wait gave up leaves, and the others' waits
// for it end the same way.  Nothing that is read from a slot is used as a memory index, and every counter still
// returns to zero.
//
// Slots, decisions and tokens cross workgroups through device-scope stores and loads (see kernels.h).
#include "kernels.h"

#include <limits.h>
#include <math.h>

namespace dreams {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr uint32_t kKeptBit = 1u << 15;  // a child's decision, beside the step's number (at most 2 * 128 steps)
constexpr uint32_t kStepMask = kKeptBit - 1;
constexpr int kArrivalShift = 53;                    // row form: a child's word: arrivals,
constexpr uint64_t kKeptWordBit = 1ull << 52;        // decision, fixed-point mass
constexpr double kFixScale = 2251799813685248.0, kFixUnit = 1.0 / kFixScale;   // 2^51 units per unit of mass

// exp(x) for x <= 0, by Tang's table-driven method: x = k ln2/256 + r with k = round(x 256/ln2) and
// |r| <= ln2/512 (ln2/256 split in two so that k times the high part is exact), e^x = 2^(k/256) e^r, with
// 2^(j/256) from a 256-entry table and e^r - 1 by its Taylor series to r^5/120 (the next term is below
// 2^-66).  Arguments below -745.5 (past the smallest subnormal) give 0.
__device__ __forceinline__ double exp_nonpos(double x, const double* tab) {
  if (!(x >= -745.5)) return 0.0;
  const double kd = rint(x * 369.3299304675746);
  const int k = (int)kd;
  double r = fma(-kd, 0x1.62e42fefp-9, x);
  r = fma(-kd, 0x1.473de6af278edp-42, r);
  const double em1 = r * fma(r, fma(r, fma(r, fma(r, 1.0 / 120.0, 1.0 / 24.0), 1.0 / 6.0), 0.5), 1.0);
  const double t = tab[k & 255];
  return ldexp(fma(t, em1, t), k >> 8);
}
// exp(d / tau) for d <= 0 as exp(d * (1 / tau)); d = 0 (the maximum itself) gives exactly 1, also where 1 / tau
// is infinite
__device__ __forceinline__ double scaled_exp(double d, double inv_tau, const double* tab) {
  return d == 0.0 ? 1.0 : exp_nonpos(d * inv_tau, tab);
}

__device__ __forceinline__ void store_d(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double load_d(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct Shared {
  double tab[256];                 // 2^(j/256)
  float wave_mt[16], wave_md[16];  // per wave: maxima and sums of a piece's statistics
  double wave_st[16], wave_sd[16];
  double wave_z[16];               // per wave: residual mass of a piece
  double scan[16];
  int pick[16], lastpos[16];
  int nsib, flag, depth;
  int par[kMaxNodes];
  int sib[kMaxNodes];
  int path[kMaxNodes];
  double rs_mt, rs_ist, rs_md, rs_isd;   // the row's merged statistics
  double st_z;                     // a child's whole residual mass ...
  int st_kept, keep_here;          // ... and decision; the decision of this piece's own token
  int fin_piece;
  double fin_before, fin_thr;
  int gave_up;                     // a wait of this workgroup reached its bound
};

// ---- wave reductions: within a row of 16 lanes by data-parallel moves (neighbours, pairs, mirrored halves), then
// the four rows in order, read into scalars: the same value in every lane, the same order on every call
template <int CTRL>
__device__ __forceinline__ int dpp(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, false);
}
constexpr int kSwap1 = 0xB1, kSwap2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140;
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __builtin_bit_cast(float, dpp<CTRL>(__builtin_bit_cast(int, x)));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)dpp<CTRL>((int)(uint32_t)u), hi = (uint32_t)dpp<CTRL>((int)(uint32_t)(u >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ float lane_of(float x, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
}
__device__ __forceinline__ double lane_of(double x, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp<kSwap1>(v));
  v = fmaxf(v, dpp<kSwap2>(v));
  v = fmaxf(v, dpp<kHalfMirror>(v));
  v = fmaxf(v, dpp<kMirror>(v));
  return fmaxf(fmaxf(lane_of(v, 0), lane_of(v, 16)), fmaxf(lane_of(v, 32), lane_of(v, 48)));
}
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp<kSwap1>(v);
  v += dpp<kSwap2>(v);
  v += dpp<kHalfMirror>(v);
  v += dpp<kMirror>(v);
  return (lane_of(v, 0) + lane_of(v, 16)) + (lane_of(v, 32) + lane_of(v, 48));
}
template <bool MAX>
__device__ __forceinline__ int wave_int(int v) {
  auto pick = [](int x, int y) { return MAX ? max(x, y) : min(x, y); };
  v = pick(v, dpp<kSwap1>(v));
  v = pick(v, dpp<kSwap2>(v));
  v = pick(v, dpp<kHalfMirror>(v));
  v = pick(v, dpp<kMirror>(v));
  return pick(pick(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
              pick(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}
// inclusive prefix over the lanes
__device__ __forceinline__ double wave_scan(double v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double o = __shfl_up(v, off);
    if (lane >= off) v += o;
  }
  return v;
}

// entries x0 + t * E + e (e < E) of a row for thread t; entries at or past x1 read as -inf
template <bool VEC, int E>
__device__ __forceinline__ void load_part(const float* row, int x0, int x1, float (&v)[E]) {
  const int base = x0 + (int)threadIdx.x * E;
  if (VEC) {   // rows are 16-byte aligned and V a multiple of 4: a vector is wholly in or out
    constexpr int W = E % 4 == 0 ? 4 : 2;
    typedef float vec __attribute__((ext_vector_type(W)));
    static_assert(E % W == 0, "whole vectors");
#pragma unroll
    for (int k = 0; k < E / W; ++k) {
      const int x = base + W * k;
      vec r;
#pragma unroll
      for (int e = 0; e < W; ++e) r[e] = -INFINITY;
      if (x < x1) r = *(const vec*)(row + x);
#pragma unroll
      for (int e = 0; e < W; ++e) v[W * k + e] = r[e];
    }
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = base + e < x1 ? row[base + e] : -INFINITY;
  }
}

// The children of node n in index order (sh.sib, sh.nsib), listed the same way by every piece; one wave.
__device__ __forceinline__ void list_children(int n, int T, const int* par, Shared& sh) {
  const int lane = threadIdx.x & 63;
  const int k0 = lane, k1 = lane + 64;
  const bool c0 = k0 > n && k0 < T && par[k0] == n;
  const bool c1 = k1 > n && k1 < T && par[k1] == n;
  const uint64_t b0 = __ballot(c0), b1 = __ballot(c1);
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  if (c0) sh.sib[__builtin_popcountll(b0 & below)] = k0;
  if (c1) sh.sib[__builtin_popcountll(b0) + __builtin_popcountll(b1 & below)] = k1;
  if (lane == 0) sh.nsib = __builtin_popcountll(b0) + __builtin_popcountll(b1);
}

// Piece j of a cluster, one row at a time.  WALK: its rows are those of a walk.  MANY: it takes more than one row.
// HOLD: a one-part piece (NT * E entries) keeps p and q in registers; else the piece's parts are streamed from memory
// in every pass over them.
template <bool VEC, bool WALK, bool MANY, bool HOLD, int NT, int E>
struct Piece {
  static constexpr int PART = NT * E, NW = NT / 64;
  // 64-bit words of a piece's slots, four each; the steps of a cluster of many rows alternate between two
  static constexpr int WORDS = 4, SLOTS = MANY ? 2 * WORDS : WORDS;
  static_assert(MANY || !WALK, "a walk takes many rows");
  static_assert(SLOTS * 8 == (MANY ? kSampledManySlotBytes : kSampledRowSlotBytes), "slot layout");
  const SampledArgs& a;
  Shared& sh;
  const int b, j, chunks;         // the sequence; this piece and the number of them
  uint32_t* const counter;        // the cluster's counter: pieces entered and (from kClusterLeft up) pieces left
  uint64_t* const slots;          // [chunks][SLOTS]
  uint32_t step = 0;
  int n = 0;                      // the row's node
  const float *trow = nullptr, *drow = nullptr;
  float lt[E], ld[E];             // (HOLD) the piece's logits ...
  double p[E], q[E];              // ... and probabilities
  double mt, inv_st, md, inv_sd;  // the row's statistics
  double C = 0.0, D = 1.0;        // the residual's state: max(p - C q, 0) / D
  double mass = 0.0;              // wave 0, lane k: piece k's part of the state's mass ...
  int src = -1;                   // ... unless it is that of child src (row form: stored by the pieces)

  // at: index of the cluster's first piece among all that have slots
  __device__ __forceinline__ Piece(const SampledArgs& args, Shared& s, int seq, int piece, int pieces, uint32_t* ctr,
                                   size_t at)
      : a(args), sh(s), b(seq), j(piece), chunks(pieces), counter(ctr), slots(args.slots + at * SLOTS) {}

  __device__ __forceinline__ bool wave0() const { return threadIdx.x < 64; }

  // Clears this piece's slots; count_in() counts it in, once they are cleared, after its first statistics.
  __device__ __forceinline__ void clear_slots() {
    if (threadIdx.x < SLOTS && chunks > 1) store_u64(slots + j * SLOTS + threadIdx.x, 0);
  }
  __device__ __forceinline__ void count_in() {
    wait_vector_memory();
    if (threadIdx.x == 0) __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  static __device__ __forceinline__ void store_u64(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // (wave 0) until ready() holds in every lane; false: the wait reached its bound
  template <typename Ready>
  __device__ __forceinline__ bool wait_until(Ready&& ready) {
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    while (true) {
      if (__ballot(!ready()) == 0) return true;
      if (__builtin_amdgcn_s_memrealtime() - t0 > a.wait_ticks) {
        if (threadIdx.x == 0) {
          raise_device_error(a.err, kErrWaitTimeout);
          sh.gave_up = 1;
        }
        return false;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  // (wave 0) one step: lane w < N stores word w of this piece, 32 + 16 bits of data; on return lane k < chunks
  // holds the words of piece k and, of the last one, the bit beside the step's number.
  template <int N>
  __device__ __forceinline__ bool exchange(uint32_t mine, uint32_t mine16, bool bit, uint32_t (&all)[N],
                                           uint32_t (&all16)[N]) {
    const int l = threadIdx.x;
    ++step;
    if (chunks == 1) {
#pragma unroll
      for (int k = 0; k < N; ++k) {
        all[k] = (uint32_t)__builtin_amdgcn_readlane((int)mine, k);
        all16[k] = (uint32_t)__builtin_amdgcn_readlane((int)mine16, k);
      }
      return bit;
    }
    const int at = MANY && step % 2 == 0 ? WORDS : 0;
    if (l < N)
      store_u64(slots + j * SLOTS + at + l, ((uint64_t)mine << 32) | ((uint64_t)mine16 << 16) | step |
                                                (l == N - 1 && bit ? kKeptBit : 0u));
    if (step == 1)   // every piece has cleared its slots
      wait_until([&] {
        return (__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & (kClusterLeft - 1)) ==
               (uint32_t)chunks;
      });
    const uint64_t* from = slots + min(l, chunks - 1) * SLOTS + at;
    bool kept = false;
    wait_until([&] {
      uint64_t w[N];
#pragma unroll
      for (int k = 0; k < N; ++k) w[k] = __hip_atomic_load(from + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      bool now = true;
#pragma unroll
      for (int k = 0; k < N; ++k) {
        now = now && ((uint32_t)w[k] & kStepMask) == step;
        all[k] = (uint32_t)(w[k] >> 32);
        all16[k] = (uint32_t)(w[k] >> 16) & 0xffffu;
      }
      kept = ((uint32_t)w[N - 1] & kKeptBit) != 0;
      return now;
    });
    return kept;
  }
  static __device__ __forceinline__ uint32_t low(double x) { return (uint32_t)__builtin_bit_cast(uint64_t, x); }
  static __device__ __forceinline__ uint32_t high(double x) { return (uint32_t)(__builtin_bit_cast(uint64_t, x) >> 32); }
  static __device__ __forceinline__ double from_words(uint32_t lo, uint32_t hi) {
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
  }

  __device__ __forceinline__ void load(int node) {
    n = node;
    const size_t row = (size_t)b * a.T + n;
    trow = a.target_logits + row * a.V;
    drow = a.draft_logits + row * a.V;
    if (HOLD) {
      const int x0 = j * PART;
      load_part<VEC>(trow, x0, min(a.V, x0 + PART), lt);
      load_part<VEC>(drow, x0, min(a.V, x0 + PART), ld);
    }
  }
  // f(e, x, target logit, draft logit) for every entry x < V of the piece, in order
  template <typename F>
  __device__ __forceinline__ void entries(F&& f) {
    const int tid = threadIdx.x, V = a.V;
    if (HOLD) {
      const int base = j * PART + tid * E;
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (base + e < V) f(e, base + e, lt[e], ld[e]);
    } else {
#pragma unroll 1
      for (int sp = 0; sp < a.sub_pieces; ++sp) {
        const long long at = ((long long)j * a.sub_pieces + sp) * PART;
        if (at >= V) break;
        const int x0 = (int)at, x1 = (int)min((long long)V, at + PART);
        float ta[E], da[E];
        load_part<VEC>(trow, x0, x1, ta);
        load_part<VEC>(drow, x0, x1, da);
        const int base = x0 + tid * E;
#pragma unroll
        for (int e = 0; e < E; ++e)
          if (base + e < V) f(e, base + e, ta[e], da[e]);
      }
    }
  }
  __device__ __forceinline__ double prob_p(float t) {
    return scaled_exp((double)t - mt, a.inv_tau, sh.tab) * inv_st;
  }
  __device__ __forceinline__ double prob_q(float d) {
    return scaled_exp((double)d - md, a.inv_tau, sh.tab) * inv_sd;
  }

  // (wave 0) sums relative to their own maxima, one pair a lane (no pair: -inf, 0), merged: the largest maximum,
  // and the sum relative to it
  __device__ __forceinline__ void merge(float& m, double& s) {
    const float top = wave_max(m);
    s = s != 0.0 ? s * scaled_exp((double)m - (double)top, a.inv_tau, sh.tab) : 0.0;
    s = wave_sum(s);
    m = top;
  }

  // The row's statistics: maxima and sums of exp((l - max) / tau), target and draft, of every wave, of the piece,
  // and of the row, and from them p and q of the piece's entries.  A one-part piece keeps its exponentials
  // relative to its wave's maxima, from which p and q follow by one factor; a streamed piece re-references each
  // thread's sums when a maximum grows.
  __device__ __forceinline__ void statistics() {
    const int tid = threadIdx.x, V = a.V, wave = tid >> 6;
    float wt = -INFINITY, wd = -INFINITY;
    double st = 0.0, sd = 0.0;
    if (HOLD) {
      const int base = j * PART + tid * E;
#pragma unroll
      for (int e = 0; e < E; ++e) {   // (entries past the vocabulary read as -inf)
        wt = fmaxf(wt, lt[e]);
        wd = fmaxf(wd, ld[e]);
      }
      wt = wave_max(wt);
      wd = wave_max(wd);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const bool in = base + e < V;
        p[e] = in ? scaled_exp((double)lt[e] - (double)wt, a.inv_tau, sh.tab) : 0.0;
        q[e] = in ? scaled_exp((double)ld[e] - (double)wd, a.inv_tau, sh.tab) : 0.0;
        st += p[e];
        sd += q[e];
      }
      st = wave_sum(st);
      sd = wave_sum(sd);
    } else {
      entries([&](int, int, float t, float d) {
        if (t > wt) {
          if (st != 0.0) st *= scaled_exp((double)wt - (double)t, a.inv_tau, sh.tab);
          wt = t;
        }
        if (d > wd) {
          if (sd != 0.0) sd *= scaled_exp((double)wd - (double)d, a.inv_tau, sh.tab);
          wd = d;
        }
        st += scaled_exp((double)t - (double)wt, a.inv_tau, sh.tab);
        sd += scaled_exp((double)d - (double)wd, a.inv_tau, sh.tab);
      });
      merge(wt, st);
      merge(wd, sd);
    }
    if ((tid & 63) == 0) {
      sh.wave_mt[wave] = wt;
      sh.wave_md[wave] = wd;
      sh.wave_st[wave] = st;
      sh.wave_sd[wave] = sd;
    }
    if (wave0() && step == 0) count_in();
    __syncthreads();
    if (wave0()) {
      float m1 = tid < NW ? sh.wave_mt[tid % NW] : -INFINITY, m2 = tid < NW ? sh.wave_md[tid % NW] : -INFINITY;
      double s1 = tid < NW ? sh.wave_st[tid % NW] : 0.0, s2 = tid < NW ? sh.wave_sd[tid % NW] : 0.0;
      merge(m1, s1);
      merge(m2, s2);
      const uint32_t mine = tid == 0   ? __builtin_bit_cast(uint32_t, m1)
                            : tid == 1 ? __builtin_bit_cast(uint32_t, m2)
                            : tid == 2 ? low(s1)
                                       : high(s1);
      const uint32_t mine16 = ((tid < 2 ? low(s2) : high(s2)) >> (tid & 1 ? 16 : 0)) & 0xffffu;
      uint32_t w[4], h[4];
      exchange<4>(mine, mine16, false, w, h);
      const bool in = tid < chunks;
      m1 = in ? __builtin_bit_cast(float, w[0]) : -INFINITY;
      m2 = in ? __builtin_bit_cast(float, w[1]) : -INFINITY;
      s1 = in ? from_words(w[2], w[3]) : 0.0;
      s2 = in ? from_words(h[0] | h[1] << 16, h[2] | h[3] << 16) : 0.0;
      const float own = m1;
      mass = s1;
      merge(m1, s1);
      merge(m2, s2);
      const double ist = 1.0 / s1;
      // piece k's share of the target's own distribution
      mass = in ? mass * scaled_exp((double)own - (double)m1, a.inv_tau, sh.tab) * ist : 0.0;
      if (tid == 0) {
        sh.rs_mt = m1;
        sh.rs_ist = ist;
        sh.rs_md = m2;
        sh.rs_isd = 1.0 / s2;
      }
    }
    __syncthreads();
    mt = sh.rs_mt;
    inv_st = sh.rs_ist;
    md = sh.rs_md;
    inv_sd = sh.rs_isd;
    if (HOLD) {
      const double ft = wt == -INFINITY ? 0.0 : scaled_exp((double)wt - mt, a.inv_tau, sh.tab) * inv_st;
      const double fd = wd == -INFINITY ? 0.0 : scaled_exp((double)wd - md, a.inv_tau, sh.tab) * inv_sd;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        p[e] *= ft;
        q[e] *= fd;
      }
    }
    C = 0.0;
    D = 1.0;
    src = -1;
  }

  // Child c (token x) of the row's node, tested against the state (C, D) its earlier siblings left, by the piece
  // that holds x; its residual mass is summed over the pieces.  Moves the state past the child.  True if c is
  // kept; the row form stores the decision (for the walk).  last: no child of the node follows.
  __device__ __forceinline__ bool test_child(int c, bool last) {
    const int tid = threadIdx.x, V = a.V, wave = tid >> 6;
    const size_t rb = (size_t)b * a.T;
    const int x = a.tokens[rb + c];
    const double CC = C + D;
    double z = 0.0, px = 0.0, qx = 0.0;
    bool holds = false;
    entries([&](int e, int xi, float t, float d) {
      const double pe = HOLD ? p[e] : prob_p(t), qe = HOLD ? q[e] : prob_q(d);
      z += fmax(pe - CC * qe, 0.0);
      if (xi == x) {
        px = pe;
        qx = qe;
        holds = true;
      }
    });
    // c's decision, by the thread holding its token (a token outside the vocabulary is never kept)
    if (holds) {
      const int keep = ((double)a.uniforms[rb + c] * qx) * D < fmax(px - C * qx, 0.0);
      if (!WALK) store_coherent(a.kept + rb + c, (int32_t)keep);
      sh.keep_here = keep;
    }
    if (!WALK && (x < 0 || x >= V) && j == 0 && tid == 0) store_coherent(a.kept + rb + c, 0);
    z = wave_sum(z);
    if ((tid & 63) == 0) sh.wave_z[wave] = z;
    __syncthreads();
    double part = mass;
    if (wave0()) {
      z = wave_sum(tid < NW ? sh.wave_z[tid % NW] : 0.0);
      const bool keep = sh.keep_here != 0;
      bool kept;
      if (WALK || chunks == 1) {
        uint32_t w[2], h[2];
        kept = exchange<2>(tid == 0 ? low(z) : high(z), 0, keep, w, h);
        kept = __ballot(kept && tid < chunks) != 0;
        part = tid < chunks ? from_words(w[0], w[1]) : 0.0;
        z = wave_sum(part);
      } else {
        if (tid == 0) store_d(a.mass + (rb + c) * chunks + j, z);
        if (last) wait_vector_memory();   // (the piece's masses are stored before its last arrival)
        // A piece's mass is at most 1 (up to rounding), a row's below 2, so that the decision's bit is free.  After
        // its wait gave up a piece's mass is meaningless and counts as 0; the others have read the statistics of
        // every piece, so theirs are parts of a sum of at most 1: none can carry into the arrivals.
        const double zc = sh.gave_up ? 0.0 : fmin(fmax(z, 0.0), 2.0);
        const uint64_t add = (1ull << kArrivalShift) + (uint64_t)rint(zc * kFixScale) + (keep ? kKeptWordBit : 0);
        uint64_t* word = (uint64_t*)(a.row_ctr + (rb + c) * a.row_stride);
        if (tid == 0) __hip_atomic_fetch_add(word, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        uint64_t v = 0;
        wait_until([&] {
          v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          return (int)(v >> kArrivalShift) == chunks;
        });
        kept = (v & kKeptWordBit) != 0;
        z = (double)(v & (kKeptWordBit - 1)) * kFixUnit;
      }
      if (tid == 0) {
        sh.keep_here = 0;
        sh.st_z = z;
        sh.st_kept = kept;
      }
    }
    __syncthreads();
    if (sh.st_z > 0.0) {
      C = CC;
      D = sh.st_z;
      mass = part;
      src = c;
    }
    return sh.st_kept;
  }

  // The token drawn if the walk ends at the row's node: the piece where the masses cross u0 times their total
  // (found alike by every piece) takes the prefix of r = max(p - C q, 0) over its entries, part by part.  -1 in
  // every other piece; the same in every thread.
  __device__ __forceinline__ int draw() {
    const int tid = threadIdx.x, V = a.V, wave = tid >> 6;
    if (wave0()) {
      if (!WALK && src >= 0 && chunks > 1)
        mass = tid < chunks ? load_d(a.mass + ((size_t)b * a.T + src) * chunks + tid) : 0.0;
      const double inc = wave_scan(mass);
      const double thr = (double)a.uniforms[(size_t)b * a.T] * lane_of(inc, 63);
      const uint64_t over = __ballot(inc > thr), some = __ballot(mass > 0.0);
      // (no crossing -- an all-zero residual: the last piece of positive mass)
      const int piece = over ? __builtin_ctzll(over) : some ? 63 - __builtin_clzll(some) : 0;
      const double before = piece > 0 ? lane_of(inc, piece - 1) : 0.0;
      if (tid == 0) {
        sh.fin_piece = piece;
        sh.fin_before = before;
        sh.fin_thr = thr;
      }
    }
    __syncthreads();
    if (sh.fin_piece != j) return -1;
    const double thr = sh.fin_thr;
    double before = sh.fin_before;
    int pick = INT_MAX, last_pos = -1;
    const int parts = HOLD ? 1 : a.sub_pieces;
    const long long first = (long long)j * parts * PART;
#pragma unroll 1
    for (int sp = 0; sp < parts && pick == INT_MAX; ++sp) {
      const long long at = first + (long long)sp * PART;
      if (at >= V) break;
      const int x0 = (int)at, x1 = (int)min((long long)V, at + PART), base = x0 + tid * E;
      float ta[E], da[E];
      if (!HOLD) {
        load_part<VEC>(trow, x0, x1, ta);
        load_part<VEC>(drow, x0, x1, da);
      }
      double r[E], own = 0.0;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        r[e] = 0.0;
        if (base + e < V) {
          const double pe = HOLD ? p[e] : prob_p(ta[e]);
          const double qe = C == 0.0 ? 0.0 : (HOLD ? q[e] : prob_q(da[e]));
          r[e] = fmax(pe - C * qe, 0.0);
        }
        own += r[e];
      }
      // the entries before this thread's, over the block in thread order
      const double inc = wave_scan(own);
      if ((tid & 63) == 63) sh.scan[wave] = inc;
      __syncthreads();
      double cum = before + (inc - own), total = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const double s = sh.scan[w];
        if (w < wave) cum += s;
        total += s;
      }
      int pk = INT_MAX, lp = -1;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        cum += r[e];
        if (pk == INT_MAX && cum > thr) pk = base + e;
        if (r[e] > 0.0) lp = base + e;
      }
      pk = wave_int<false>(pk);
      lp = wave_int<true>(lp);
      if ((tid & 63) == 0) {
        sh.pick[wave] = pk;
        sh.lastpos[wave] = lp;
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        pick = min(pick, sh.pick[w]);
        last_pos = max(last_pos, sh.lastpos[w]);
      }
      before += total;
      __syncthreads();
    }
    // (rounding between the piece masses and this prefix can leave the crossing just outside the piece: then
    // the piece's last entry of positive mass)
    if (pick == INT_MAX) pick = last_pos >= 0 ? last_pos : (int)min((long long)V - 1, first);
    return pick;
  }

  // (thread 0, once this piece's stores are done) counts this piece out; true in the cluster's last one
  __device__ __forceinline__ bool leave() {
    return __hip_atomic_fetch_add(counter, kClusterLeft, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) / kClusterLeft ==
           (uint32_t)(chunks - 1);
  }
};

// ---------------------------------------------------------------------------------------------- row form
// The walk over every node's decisions and prepared token, by the sequence's last row to finish.
__device__ void walk_decisions(const SampledArgs& a, int b, Shared& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int T = a.T;
  const size_t rb = (size_t)b * T;
  if (wave == 0) {
    // lane l holds nodes l and l + 64; the first kept child of each node, from the root
    int par_h[2], kept_h[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = lane + 64 * h;
      par_h[h] = i < T ? a.parent[rb + i] : -1;
      kept_h[h] = i > 0 && i < T ? load_coherent(a.kept + rb + i) : 0;
    }
    int node = 0, depth = 0;
    if (lane == 0) sh.path[0] = 0;
    while (true) {
      const uint64_t k0 = __ballot(kept_h[0] && par_h[0] == node && lane > node);
      const uint64_t k1 = __ballot(kept_h[1] && par_h[1] == node && lane + 64 > node);
      if ((k0 | k1) == 0) break;
      node = k0 ? __builtin_ctzll(k0) : 64 + __builtin_ctzll(k1);
      ++depth;
      if (lane == 0) sh.path[depth] = node;
    }
    if (lane == 0) {
      a.accept_len[b] = depth;
      a.next_token[b] = load_coherent(a.final_token + rb + node);
      reset_counter(a.seq_ctr + b);
      sh.depth = depth;
    }
  }
  __syncthreads();
  const int depth = sh.depth;
  if (tid < T) {
    a.accept_path[rb + tid] = tid <= depth ? sh.path[tid] : -1;
    uint32_t* words = a.row_ctr + (rb + tid) * a.row_stride;
    __hip_atomic_store((uint64_t*)words, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    reset_counter(words + kSampledRowCounter);
  }
}

// Row n (loaded, its children listed): its children's decisions, and the token emitted if the walk ends there.
template <typename P>
__device__ __forceinline__ void take_row(const SampledArgs& a, Shared& sh, P& pc, int b, int n) {
  pc.statistics();
  const int nsib = sh.nsib;
  for (int k = 0; k < nsib && !sh.gave_up; ++k) pc.test_child(sh.sib[k], k == nsib - 1);
  const int pick = pc.draw();
  if (pick >= 0 && threadIdx.x == 0) store_coherent(a.final_token + (size_t)b * a.T + n, pick);
}
// The piece has taken its cluster's rows.
template <typename P>
__device__ __forceinline__ void rows_done(const SampledArgs& a, Shared& sh, P& pc, int b) {
  // Every piece counts itself out once its decisions and tokens are stored; the cluster's last piece counts it as
  // done, and the sequence's last cluster runs the walk.
  wait_vector_memory();
  __syncthreads();
  if (threadIdx.x == 0)
    sh.flag = pc.leave() && __hip_atomic_fetch_add(a.seq_ctr + b, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                                (uint32_t)(a.clusters - 1);
  __syncthreads();
  if (sh.flag) walk_decisions(a, b, sh);
}

__device__ __forceinline__ uint32_t* row_counter(const SampledArgs& a, int b, int n) {
  return a.row_ctr + ((size_t)b * a.T + n) * a.row_stride + kSampledRowCounter;
}

// Workgroup (b, n, j): piece j of row n.
template <bool VEC, int NT, int E>
__global__ __launch_bounds__(NT) void tree_accept_sampled_rows_kernel(SampledArgs a) {
  __shared__ Shared sh;
  const int tid = threadIdx.x, T = a.T;
  const int j = (int)(blockIdx.x % (unsigned)a.chunks), row = (int)(blockIdx.x / (unsigned)a.chunks);
  const int b = row / T, n = row - b * T;
  Piece<VEC, false, false, true, NT, E> pc(a, sh, b, j, a.chunks, row_counter(a, b, n), (size_t)row * a.chunks);
  pc.clear_slots();
  pc.load(n);
  if (tid < 256) sh.tab[tid] = exp2((double)tid * (1.0 / 256.0));
  if (tid < 64) list_children(n, T, a.parent + (size_t)b * T, sh);
  if (tid == 0) sh.gave_up = sh.keep_here = 0;
  __syncthreads();
  take_row(a, sh, pc, b, n);
  rows_done(a, sh, pc, b);
}

// --------------------------------------------------------------------------------------------- walk form
// Piece j of the cluster that walks sequence b, its first row loaded: every row that the walk visits, from the root.
template <typename P>
__device__ __forceinline__ void walk_rows(const SampledArgs& a, Shared& sh, P& pc, int b, int j) {
  const int tid = threadIdx.x, T = a.T;
  const size_t rb = (size_t)b * T;
  int depth = 0;
  for (int node = 0;;) {
    if (tid < 64) list_children(node, T, sh.par, sh);
    pc.statistics();
    const int nsib = sh.nsib;
    int next = -1;
    for (int k = 0; k < nsib && next < 0 && !sh.gave_up; ++k) {
      const int c = sh.sib[k];
      if (pc.test_child(c, k == nsib - 1)) next = c;
    }
    if (next < 0 || sh.gave_up) break;
    node = next;
    ++depth;
    if (tid == 0) sh.path[depth] = node;
    pc.load(node);
    __syncthreads();   // every thread has read this node's children and whether a wait gave up
  }
  const int pick = pc.draw();
  if (pick >= 0 && tid == 0) a.next_token[b] = pick;
  if (j == 0) {
    if (tid < T) a.accept_path[rb + tid] = tid <= depth ? sh.path[tid] : -1;
    if (tid == 0) a.accept_len[b] = depth;
  }
  wait_vector_memory();
  __syncthreads();
  if (tid == 0 && pc.leave()) reset_counter(a.seq_ctr + b);
}

__device__ __forceinline__ void start_walk(const SampledArgs& a, Shared& sh, int b) {
  const int tid = threadIdx.x;
  if (tid < 256) sh.tab[tid] = exp2((double)tid * (1.0 / 256.0));
  if (tid < a.T) sh.par[tid] = a.parent[(size_t)b * a.T + tid];
  if (tid == 0) {
    sh.gave_up = sh.keep_here = 0;
    sh.path[0] = 0;
  }
  __syncthreads();
}

// Workgroup (b, j): piece j of sequence b's walk.
template <bool VEC, bool HOLD, int NT, int E>
__global__ __launch_bounds__(NT) void tree_accept_sampled_walk_kernel(SampledArgs a) {
  __shared__ Shared sh;
  const int b = (int)(blockIdx.x / (unsigned)a.chunks), j = (int)(blockIdx.x % (unsigned)a.chunks);
  Piece<VEC, true, true, HOLD, NT, E> pc(a, sh, b, j, a.chunks, a.seq_ctr + b, (size_t)b * a.chunks);
  pc.clear_slots();
  pc.load(0);
  start_walk(a, sh, b);
  walk_rows(a, sh, pc, b, j);
}

// ------------------------------------------------------------------------------------------- either form
// Whether some path from the root has more than `most` nodes, breadth-first over ballots (lane l holds nodes l and
// l + 64); the same in every wave.
__device__ __forceinline__ bool path_longer_than(const int* par, int T, int most) {
  const int lane = threadIdx.x & 63;
  const int p0 = lane < T ? par[lane] : -1, p1 = lane + 64 < T ? par[lane + 64] : -1;
  const bool v0 = p0 >= 0 && p0 < lane, v1 = p1 >= 0 && p1 < lane + 64;
  uint64_t s0 = 1, s1 = 0;   // the nodes at this depth
  for (int nodes = 1; (s0 | s1) != 0; ++nodes) {
    if (nodes > most) return true;
    const bool n0 = v0 && (s0 >> p0 & 1) != 0;
    const bool n1 = v1 && ((p1 < 64 ? s0 >> p1 : s1 >> (p1 - 64)) & 1) != 0;
    s0 = __ballot(n0);
    s1 = __ballot(n1);
  }
  return false;
}

// First a workgroup per piece of every sequence's walk (EW entries a thread), which leave where the tree has longer
// paths; then workgroups (c, b, j), piece j (ER entries a thread) of sequence b's cluster c, which takes rows c,
// c + clusters, ..., and leave where it has not.  A sequence's walk has the slots of its clusters.
// (At most 128 registers a lane: parts of 10240 entries, vocabularies of 524289 to 655360, spill five; 8 kept drafts of
// 600000 47 us, 101 before there was a walk.)
template <bool VEC, bool HOLD, int NT, int EW, int ER>
__global__ __launch_bounds__(NT, 4) void tree_accept_sampled_either_kernel(SampledArgs a) {
  __shared__ Shared sh;
  const int n = (int)blockIdx.x, walkers = a.B * a.walk_chunks;
  if (n < walkers) {
    const int b = n / a.walk_chunks, j = n - b * a.walk_chunks;
    Piece<VEC, true, true, HOLD, NT, EW> pc(a, sh, b, j, a.walk_chunks, a.seq_ctr + b,
                                            (size_t)b * a.clusters * a.chunks);
    pc.load(0);
    start_walk(a, sh, b);
    if (path_longer_than(sh.par, a.T, a.max_visits)) return;
    pc.clear_slots();
    walk_rows(a, sh, pc, b, j);
    return;
  }
  const int r = (n - walkers) / a.chunks, j = n - walkers - r * a.chunks;
  const int c = r / a.B, b = r - c * a.B;
  Piece<VEC, false, true, HOLD, NT, ER> pc(a, sh, b, j, a.chunks, row_counter(a, b, c),
                                           ((size_t)b * a.clusters + c) * a.chunks);
  start_walk(a, sh, b);
  if (!path_longer_than(sh.par, a.T, a.max_visits)) return;
  pc.clear_slots();
  for (int row = c; row < a.T; row += a.clusters) {
    pc.load(row);
    if (threadIdx.x < 64) list_children(row, a.T, sh.par, sh);
    take_row(a, sh, pc, b, row);
    if (sh.gave_up) break;
  }
  rows_done(a, sh, pc, b);
}

}  // namespace

hipError_t launch_tree_accept_sampled(const SampledArgs& a, hipStream_t stream) {
  if (a.chunks > kSampledMaxPieces) return hipErrorInvalidValue;
  const long long grid = (long long)a.B * ((long long)a.clusters * a.chunks + a.walk_chunks);
  auto go = [&](auto kern, int threads) {
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(threads), 0, stream, a);
    return hipGetLastError();
  };
  if (a.form == kSampledRows)
    return a.vec4 ? go(tree_accept_sampled_rows_kernel<true, 512, 8>, 512)
                  : go(tree_accept_sampled_rows_kernel<false, 512, 8>, 512);
#define DREAMS_EITHER(HOLD, NT, EW, ER)                                               \
  return a.vec4 ? go(tree_accept_sampled_either_kernel<true, HOLD, NT, EW, ER>, NT)   \
                : go(tree_accept_sampled_either_kernel<false, HOLD, NT, EW, ER>, NT)
  if (a.form == kSampledEither) {
    if (a.sub_pieces > 1) DREAMS_EITHER(false, 1024, 8, 8);
    switch (a.part) {
      case 2048: DREAMS_EITHER(true, 512, 4, 8);
      case 4096: DREAMS_EITHER(true, 512, 8, 8);
      case 8192: DREAMS_EITHER(true, 1024, 8, 8);
      case 10240: DREAMS_EITHER(true, 1024, 10, 10);
    }
    return hipErrorInvalidValue;
  }
#undef DREAMS_EITHER
#define DREAMS_WALK(HOLD, NT, E)                                                        \
  return a.vec4 ? go(tree_accept_sampled_walk_kernel<true, HOLD, NT, E>, NT)            \
                : go(tree_accept_sampled_walk_kernel<false, HOLD, NT, E>, NT)
  if (a.sub_pieces > 1) DREAMS_WALK(false, 1024, 8);
  switch (a.part) {
    case 2048: DREAMS_WALK(true, 512, 4);
    case 4096: DREAMS_WALK(true, 1024, 4);
    case 8192: DREAMS_WALK(true, 1024, 8);
    case 10240: DREAMS_WALK(true, 1024, 10);
  }
#undef DREAMS_WALK
  return hipErrorInvalidValue;
}

}  // namespace dreams
