// Greedy tree acceptance (the paper's Section 2, "Speculative decoding": drafts are kept while they equal the
// target's own token at their position; at the first mismatch the target's token replaces the draft).
//
// One kernel, bound by HBM on the logits (B*T*V*4 bytes, the only large input).  Each (sequence, node) row of V
// logits is cut into `chunks` pieces, one 256-thread workgroup per piece.  A thread loads four 16-byte vectors at a
// time and has the next four in flight while it compares them, so that a workgroup streams a piece of any
// length: with one piece per row in large batches, its start and its arrival below are paid once per row
// (16 x 128 x 152064: 193 us, 6.45 TB/s, against 213 us with a burst of 32 loads a thread per 32768 logits; an odd
// vocabulary, whose rows start at any word, takes the same vectors between single entries at the ends:
// 16 x 100 x 30001 45.4 -> 39 us).  The loads carry the non-temporal hint: each byte is read once.  A workgroup
// publishes its piece's best (value, index) and arrives at its sequence's counters; the last workgroup of the
// sequence to arrive merges all of the sequence's pieces and runs the path scan:
//   * piece best: ties go to the smallest index -- every thread visits its elements in increasing order and
//     replaces its candidate only on a strictly larger value, and every merge prefers the smaller index on
//     equal values (fp32 comparison, so -0.0 and +0.0 are equal);
//   * arrival: a sequence's workgroups are dealt round-robin to up to 8 group counters (each on a cache line
//     of its own where the counter region allows), and the last arrival of each group arrives at the
//     sequence counter, so that no counter takes more than a few dozen atomics (atomics on one line
//     serialise);
//   * path scan: one wave sweeps the tree from the root, one depth per round, growing the set of consistent
//     nodes (every draft on the way equal to the target's token at its parent) by ballots; the last round's
//     smallest new member is the deepest consistent node (smallest index among equals).
// The pieces travel through device-scope stores and loads (see kernels.h); the tree (tokens, parents) is
// fetched by every workgroup at entry, ahead of its logits, for whichever one ends up finishing the sequence.
#include "accept_scan.h"
#include "kernels.h"

#include <limits.h>
#include <math.h>

namespace dreams {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// true iff (v2, i2) beats (v1, i1): larger value, or equal value and smaller index
__device__ __forceinline__ bool better(float v2, int i2, float v1, int i1) {
  return v2 > v1 || (v2 == v1 && i2 < i1);
}

// Block-wide best (value, index); the result is valid in every thread.
__device__ __forceinline__ void block_best(float& v, int& i, float* red_v, int* red_i) {
  constexpr int NW = kAcceptThreads / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const float v2 = __shfl_xor(v, off);
    const int i2 = __shfl_xor(i, off);
    if (better(v2, i2, v, i)) { v = v2; i = i2; }
  }
  __syncthreads();   // earlier readers of red_v / red_i are done
  if (lane == 0) { red_v[wave] = v; red_i[wave] = i; }
  __syncthreads();
  v = red_v[0];
  i = red_i[0];
#pragma unroll
  for (int w = 1; w < NW; ++w)
    if (better(red_v[w], red_i[w], v, i)) { v = red_v[w]; i = red_i[w]; }
}

constexpr int U = 4;   // 16-byte vectors a thread loads at a time

__global__ __launch_bounds__(kAcceptThreads) void tree_accept_kernel(AcceptArgs a) {
  constexpr int NT = kAcceptThreads, NW = NT / 64, STEP = NT * 4;
  __shared__ float red_v[NW];
  __shared__ int red_i[NW];
  __shared__ int flag;
  __shared__ int am_s[kMaxNodes], tok_s[kMaxNodes], par_s[kMaxNodes];

  const int tid = threadIdx.x, wave = tid >> 6;
  const int T = a.T;
  const int n = blockIdx.x;                 // ((b * T) + i) * chunks + c
  const int per_seq = T * a.chunks;         // workgroups of one sequence
  const int b = n / per_seq, local = n - b * per_seq;
  const int bi = n / a.chunks, c = n - bi * a.chunks;
  int tok_r = 0, par_r = 0;
  if (tid < T) {
    tok_r = a.tokens[(size_t)b * T + tid];
    par_r = a.parent[(size_t)b * T + tid];
  }
  const float* row = a.logits + (size_t)bi * a.V;
  const int x0 = c * a.chunk, x1 = min(a.V, x0 + a.chunk);

  // ---- best (value, index) of this piece: whole 16-byte vectors [xa, xe) of the row, wherever it starts, between
  // at most three single entries at either end.  Each thread visits its entries in increasing order.
  float bv = -INFINITY;
  int bx = INT_MAX;
  auto visit = [&](float v, int x) {
    if (v > bv || bx == INT_MAX) { bv = v; bx = x; }
  };
  const int xa = min(x1, x0 + (int)(-(((uintptr_t)(row + x0)) >> 2) & 3));
  const int xe = xa + ((x1 - xa) & ~3);
  if (x0 + tid < xa) visit(row[x0 + tid], x0 + tid);
  if (xa < xe) {
    // U vectors a thread at a time, the next U in flight while these are compared; the loads are unconditional
    // (clamped to the last vector), so that all of a batch are in flight together
    auto load = [&](f32x4 (&r)[U], int xb) {
#pragma unroll
      for (int u = 0; u < U; ++u) r[u] = __builtin_nontemporal_load((const f32x4*)(row + min(xb + u * STEP, xe - 4)));
    };
    auto compare = [&](const f32x4 (&r)[U], int xb) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int x = xb + u * STEP;
        if (x < xe) {
#pragma unroll
          for (int e = 0; e < 4; ++e) visit(r[u][e], x + e);
        }
      }
    };
    f32x4 r0[U], r1[U];
    int xb = xa + tid * 4;
    load(r0, xb);
    for (int left = xe - xa; left > 0; left -= 2 * U * STEP, xb += 2 * U * STEP) {   // (block-uniform)
      if (left > U * STEP) load(r1, xb + U * STEP);
      compare(r0, xb);
      if (left > 2 * U * STEP) load(r0, xb + 2 * U * STEP);
      if (left > U * STEP) compare(r1, xb + U * STEP);
    }
  }
  if (xe + tid < x1) visit(row[xe + tid], xe + tid);
  block_best(bv, bx, red_v, red_i);

  // ---- publish it and arrive: group counter, then (last of the group) the sequence counter
  if (tid == 0) {
    store_coherent(a.part_val + n, bv);
    store_coherent(a.part_idx + n, bx);
    wait_vector_memory();
    const int NG = a.groups;
    const int g = local % NG;
    uint32_t* gc = a.counters + a.group_base + ((size_t)b * NG + g) * a.group_stride;
    bool last = arrive_last(gc, (uint32_t)((per_seq - g + NG - 1) / NG));
    if (last) {
      reset_counter(gc);   // every workgroup of the group has arrived: ready for the next call
      last = arrive_last(a.counters + b, (uint32_t)NG);
    }
    flag = last;
  }
  __syncthreads();
  if (!flag) return;

  // ---- the sequence's last workgroup: every row's argmax from its pieces (all loads of a batch of 8 pieces
  // in flight together, merged in piece order), then the path scan
  if (tid < T) {
    float v = -INFINITY;
    int x = INT_MAX;
    const size_t p0 = ((size_t)b * T + tid) * a.chunks;
    for (int c0 = 0; c0 < a.chunks; c0 += 8) {
      float pv[8];
      int px[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const size_t pp = p0 + min(c0 + k, a.chunks - 1);
        pv[k] = load_coherent(a.part_val + pp);
        px[k] = load_coherent(a.part_idx + pp);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (c0 + k < a.chunks && better(pv[k], px[k], v, x)) { v = pv[k]; x = px[k]; }
    }
    am_s[tid] = x;
    tok_s[tid] = tok_r;
    par_s[tid] = par_r;
  }
  if (tid == 0) reset_counter(a.counters + b);   // ready for the next call
  __syncthreads();
  if (a.target_argmax && tid < T) a.target_argmax[(size_t)b * T + tid] = am_s[tid];
  if (wave != 0) return;

  path_scan_wave(am_s, tok_s, par_s, T, a.accept_len + b, a.accept_path + (size_t)b * T, a.next_token + b);
}

}  // namespace

hipError_t launch_tree_accept(const AcceptArgs& a, hipStream_t stream) {
  const int grid = a.B * a.T * a.chunks;
  hipLaunchKernelGGL(tree_accept_kernel, dim3(grid), dim3(kAcceptThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace dreams
