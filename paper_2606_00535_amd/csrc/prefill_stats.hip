// Attention statistics of a prompt's own causal attention (the prefilling pass), where the paper reads them:
// AE(l) of Section 3.2 averages the entropy of a layer's attention rows over the n prompt tokens, and Eq. 2 of
// Section 3.1 scores the visual tokens with the final layer's attention of the prefill.  Row i of query head h
// attends the prompt's slots 0..i (the decoder's causal mask):
//     lse[h,i]     = log sum_{j <= i} exp(scale * q_i . k_j)
//     entropy[h,i] = -sum_{j <= i} A[h,i,j] log A[h,i,j],   A[h,i,j] = exp(scale * q_i . k_j - lse[h,i]).
// No value product is needed, so this is half of a causal attention forward.
//
//   * prefill_stats_kernel: a workgroup of 8 waves owns 128 or 256 query rows of one query head; a wave owns 32
//     rows as two 16-row matrix-core B operands (its queries stay in registers).  The prompt's keys 0 .. the
//     workgroup's last row stream through an LDS ring of 64-key stages (LDS-DMA copies, several stages ahead); of
//     128 rows, four waves take each stage's first 32 keys, four its second 32 (their states meet in LDS at the
//     end): S^T = K Q^T on v_mfma_f32_16x16x32_bf16 with the key rows as the A operand.
//     Each lane keeps, for each of its 2 rows, an online (reference, sum, entropy term) over the keys its
//     quad sees, in log2 units; the reference only moves when a score passes it by more than 2^8 (the sums
//     stay finite and the statistics do not depend on it), and the four quads are merged at the end.  Only
//     32-key blocks that cross the diagonal or the prompt's end are masked, in a loop of their own (in one loop
//     the two paths' states met in register copies).  Workgroups are ordered so that the row blocks with the
//     most keys start first; a single round's second half takes them in the opposite order.
//     What bounds it is the vector ALU (active in 74 % of the cycles a compute unit is busy: per score an fma, an
//     exp2 at a quarter rate, an add and an fma, beside a quarter of a matrix instruction), as long as every compute unit holds two
//     workgroups to the end: with few workgroups, 256-row ones leave the longest alone with two waves a SIMD.  3136 rows x 32
//     heads x 128: 85 us as 256-row workgroups, 72 us as 128-row ones, 63 us with the masked blocks apart, the
//     maxima as three-input chains and the reference test on unscaled products (kernel times).
//   * prefill_entropy_mean_kernel: one workgroup, the fp64 mean of the prompt rows' entropies over every head
//     and sequence (rows i >= n_b hold 0 and do not count).
#include "kernels.h"

#include <math.h>

namespace dreams {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8;
constexpr int kRB = 2;                        // 16-row blocks per wave
constexpr int kRowsPerWave = 16 * kRB;
constexpr int kRowsPerWgMax = kRowsPerWave * kWaves;   // over the key groups (see below)
constexpr int kKeys = 64;                     // keys per ring stage
constexpr int kStages = 4;                    // ring stages
constexpr float kLazyLog2 = 8.0f;             // slack of the reference before it moves

// Key rows in LDS: rows of D bf16, the 16-byte chunk c of row r at position c ^ swz(r), which puts the 16 rows
// of one operand read (rows (m%4)*4 + m/4 of a 16-row block, one chunk) on distinct banks.
template <int D>
struct KRows {
  static constexpr int ROW = D * 2, CPR = D / 8, RPL = 256 / ROW;
  static __device__ __forceinline__ int swz(int r) {
    if constexpr (D == 128) return ((r >> 2) & 3) * 4 + (r & 1) * 2 + 1;
    return (r / RPL) % CPR;
  }
  static __device__ __forceinline__ int off(int r, int c) { return r * ROW + ((c ^ swz(r)) << 4); }
};

typedef __attribute__((address_space(3))) void lds_void;
__device__ __forceinline__ uint32_t lds_addr(const void* p) { return (uint32_t)(uintptr_t)(lds_void*)p; }
// wave-wide 16-byte copy into LDS: lane l's 16 bytes land at m0 + 16 l (m0 wave-uniform)
__device__ __forceinline__ void copy16_to_lds(uint32_t m0, const void* src) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(m0), "v"(src) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// 16-byte load into registers, issued like the copies (so that a wait for it can leave later copies in flight)
__device__ __forceinline__ void load16(bf16x8& dst, const void* src) {
  asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(dst) : "v"(src) : "memory");
}
// at most N vector-memory operations of this wave outstanding; the registers loaded before them are tied to the
// wait (one statement for all of them, so that no use or copy of any is scheduled ahead of it)
template <int N>
__device__ __forceinline__ void wait_vm_tied(bf16x8 (&x)[4]) {
  asm volatile("s_waitcnt vmcnt(%4)" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]) : "n"(N) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vm_tied(bf16x8 (&x)[2][4]) {
  asm volatile("s_waitcnt vmcnt(%8)"
               : "+v"(x[0][0]), "+v"(x[0][1]), "+v"(x[0][2]), "+v"(x[0][3]), "+v"(x[1][0]), "+v"(x[1][1]),
                 "+v"(x[1][2]), "+v"(x[1][3])
               : "n"(N)
               : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vm_tied(bf16x8 (&x)[2][2]) {
  asm volatile("s_waitcnt vmcnt(%4)" : "+v"(x[0][0]), "+v"(x[0][1]), "+v"(x[1][0]), "+v"(x[1][1]) : "n"(N) : "memory");
}
// at most k * PER of this wave's copies outstanding (k <= K)
template <int PER, int K>
__device__ __forceinline__ void wait_vm_steps(int k) {
  if constexpr (K > 0) {
    if (k >= K) {
      wait_vm<PER * K>();
      return;
    }
    wait_vm_steps<PER, K - 1>(k);
  } else {
    wait_vm<0>();
  }
}
// workgroup barrier once this wave's LDS accesses are done; copies stay in flight
__device__ __forceinline__ void barrier_lds() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// A state (m, l, e) in log2 units: l = sum 2^(z-m), e = sum 2^(z-m) (z-m).  Re-referenced to M with weight
// w = 2^(m-M): l -> w l, e -> w (e + (m-M) l).
__device__ __forceinline__ void rescale(float& m, float& l, float& e, float M) {
  if (m == M) return;
  const float w = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M);
  e = w == 0.f ? 0.f : w * fmaf(m - M, l, e);
  l *= w;
  m = M;
}

// KG key groups: each takes its part of every stage, with kWaves / KG of the waves
template <int D, int KG>
__global__ __launch_bounds__(64 * kWaves, 2) void prefill_stats_kernel(PrefillArgs a) {
  using L = KRows<D>;
  constexpr int kRowsPerWg = kRowsPerWgMax / KG, kRowWaves = kWaves / KG, KPG = kKeys / KG;
  static_assert(KG == 1 || KG == 2, "one or two 32-key halves of a stage per group");
  constexpr int DS = D / 32;
  constexpr int STAGE = kKeys * L::ROW;          // bytes of a stage
  constexpr int CPW = STAGE / 1024 / kWaves;     // wave-wide 1 KB copies per wave per stage
  static_assert(CPW >= 1 && CPW * 1024 * kWaves == STAGE, "copy split");
  extern __shared__ __attribute__((aligned(1024))) unsigned char ring[];   // kStages x STAGE
  // Workgroup order: row blocks with the most keys first; if they all fit two to a compute unit, those beyond the
  // first of each (which share a compute unit with one of the first) take the blocks in the opposite order, so
  // that the longest block is paired with the shortest.
  const int nblk = (a.N + kRowsPerWg - 1) / kRowsPerWg, BH = a.B * a.Hq;
  const int n = blockIdx.x, W = gridDim.x;
  const int rank = (n >= a.cus && W <= 2 * a.cus) ? W - 1 - (n - a.cus) : n;
  const int blk = nblk - 1 - rank / BH;
  const int bh = rank - (rank / BH) * BH;
  const int h = bh % a.Hq, b = bh / a.Hq;
  const int g = h / a.G;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, quad = lane >> 4;
  int nb = __builtin_amdgcn_readfirstlane(a.prompt_len[b]);
  nb = nb < 0 ? 0 : (nb > a.N ? a.N : nb);

  const int r0 = blk * kRowsPerWg;                  // the workgroup's first row
  const int kgrp = wave / kRowWaves;                // the wave's part of every stage
  const int rw0 = r0 + (wave % kRowWaves) * kRowsPerWave;   // the wave's first row
  const size_t qrow0 = ((size_t)b * a.Hq + h) * a.N;
  const unsigned char* kbase = (const unsigned char*)a.k + ((size_t)b * a.Hkv + g) * a.S_cap * L::ROW;
  const int kend = min(r0 + kRowsPerWg, nb);        // keys any live row of the workgroup can see
  const int nst = kend > 0 ? (kend + kKeys - 1) / kKeys : 0;
  const uint32_t ring_lds = __builtin_amdgcn_readfirstlane(lds_addr(ring));

  // copies of stage st: 1 KB block ci = wave * CPW + j; lane l brings row r = (ci * 1024 + 16 l) / ROW of the
  // stage, position l % CPR, i.e. the key row's chunk (l % CPR) ^ swz(r); rows past the cache repeat its last
  auto issue = [&](int st) {
    const uint32_t dst = __builtin_amdgcn_readfirstlane(ring_lds + (st % kStages) * STAGE);
#pragma unroll
    for (int j = 0; j < CPW; ++j) {
      const int ci = wave * CPW + j;
      const int e = ci * 64 + lane;
      const int r = e / L::CPR, p = e - r * L::CPR;
      const int key = min(st * kKeys + r, a.S_cap - 1);
      copy16_to_lds(dst + ci * 1024, kbase + (size_t)key * L::ROW + ((p ^ L::swz(r)) << 4));
    }
  };
  // queries first (registers), then the first stages' copies; the wait for the queries leaves those in flight
  bf16x8 qf[kRB][DS];
  const unsigned char* qbase = (const unsigned char*)a.q + qrow0 * L::ROW;
#pragma unroll
  for (int rb = 0; rb < kRB; ++rb) {
    const int row = min(rw0 + rb * 16 + col, a.N - 1);
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) load16(qf[rb][ds], qbase + (size_t)row * L::ROW + (ds * 32 + quad * 8) * 2);
  }
  // always kStages - 1 stages (past the last one they repeat it, unread), so that the wait count is fixed
  for (int st = 0; st < kStages - 1; ++st) issue(min(st, max(nst - 1, 0)));
  wait_vm_tied<(kStages - 1) * CPW>(qf);
  // scores are scaled by c = |scale| log2(e) inside the exponent; a negative scale flips the queries' signs
  // (exact in bf16)
  const float c = fabsf(a.scale_log2);
  if (a.scale_log2 < 0.f) {
#pragma unroll
    for (int rb = 0; rb < kRB; ++rb)
#pragma unroll
      for (int ds = 0; ds < DS; ++ds) qf[rb][ds] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, qf[rb][ds]) ^ 0x80008000u);
  }

  float m[kRB], l[kRB], e[kRB];
  float thr[kRB];   // the products past which the reference moves: (m + kLazyLog2) / c, kept up by the plain blocks
#pragma unroll
  for (int rb = 0; rb < kRB; ++rb) {
    m[rb] = thr[rb] = -INFINITY;
    l[rb] = 0.f;
    e[rb] = 0.f;
  }
  const int ka_row = (col & 3) * 4 + (col >> 2);   // A row m holds key kb*16 + (m%4)*4 + m/4
  const int wlast = min(rw0 + kRowsPerWave, nb) - 1;   // the wave's last live row (< rw0: none)

  // 32 keys of a stage, its first or second half (two 16-key blocks): lane (col, quad) gets keys kk0 + 16 kb + 4 t + quad
  // (t = 0..3) of rows rw0 + 16 rb + col.
  auto products = [&](f32x4 (&s)[kRB][2], const unsigned char* tile, int half) {
    bf16x8 kf[2][DS];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int ds = 0; ds < DS; ++ds)
        kf[kb][ds] = *(const bf16x8*)(tile + L::off((half * 2 + kb) * 16 + ka_row, ds * 4 + quad));
#pragma unroll
    for (int ds = 0; ds < DS; ++ds)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int rb = 0; rb < kRB; ++rb)
          s[rb][kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kb][ds], qf[rb][ds],
                                                              ds == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : s[rb][kb], 0, 0, 0);
  };
  // every key visible: the reference moves (rarely) when a score passes it by more than 2^8, then each score costs
  // one fma, one exp2, one add and one fma
  auto plain_block = [&](const f32x4 (&s)[kRB][2]) {
    float smax[kRB];
    bool grow = false;
#pragma unroll
    for (int rb = 0; rb < kRB; ++rb) {
      // (a chain, so that every step is one three-input maximum)
      float x = vmax(vmax(s[rb][0][0], s[rb][0][1]), s[rb][0][2]);
      x = vmax(vmax(x, s[rb][0][3]), s[rb][1][0]);
      x = vmax(vmax(x, s[rb][1][1]), s[rb][1][2]);
      smax[rb] = vmax(x, s[rb][1][3]);
      grow |= smax[rb] > thr[rb];
    }
    if (__any(grow)) {
#pragma unroll
      for (int rb = 0; rb < kRB; ++rb)
        if (smax[rb] > thr[rb]) {
          rescale(m[rb], l[rb], e[rb], c * smax[rb]);
          thr[rb] = (m[rb] + kLazyLog2) / c;
        }
    }
#pragma unroll
    for (int rb = 0; rb < kRB; ++rb) {
      float ps, es;   // (the block among itself first: fewer roundings at the sums' size)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float d = fmaf(s[rb][kb][t], c, -m[rb]);
          const float p = __builtin_amdgcn_exp2f(d);
          ps = kb + t == 0 ? p : ps + p;
          es = kb + t == 0 ? p * d : fmaf(p, d, es);
        }
      l[rb] += ps;
      e[rb] += es;
    }
  };
  // blocks that cross the diagonal or the prompt's end
  auto edge_block = [&](const f32x4 (&s)[kRB][2], int kk0) {
#pragma unroll
    for (int rb = 0; rb < kRB; ++rb) {
      float z[2][4], zmax = -INFINITY;
      const int row = rw0 + rb * 16 + col;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int key = kk0 + kb * 16 + 4 * t + quad;
          z[kb][t] = (key > row || key >= nb) ? -INFINITY : s[rb][kb][t] * c;
        }
        zmax = vmax(zmax, vmax(vmax(z[kb][0], z[kb][1]), vmax(z[kb][2], z[kb][3])));
      }
      if (zmax > m[rb] + kLazyLog2) rescale(m[rb], l[rb], e[rb], zmax);
      if (m[rb] != -INFINITY) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const float d = fmaxf(z[kb][t] - m[rb], -1.0e4f);   // (a masked key: p = 0 and a zero term)
            const float p = __builtin_amdgcn_exp2f(d);
            l[rb] += p;
            e[rb] = fmaf(p, d, e[rb]);
          }
      }
    }
  };

  auto next_stage = [&](int st) {
    // this wave's copies of stage st have landed (the later stages it issued may still be in flight)
    wait_vm_steps<CPW, kStages - 2>(min(nst, max(st + kStages - 1, kStages - 1)) - st - 1);
    barrier_lds();   // stage st complete for every wave; every wave is past stage st - 1, whose slot is free
    if (st + kStages - 1 < nst) issue(st + kStages - 1);
  };
  // The wave's plain stages come first, then those it masks, then those that no live row of it sees; every wave
  // passes every stage's barrier, in whichever loop.
  const int first = kgrp * KPG;   // the wave's first key of a stage
  const int lim = min(rw0, nb - 1) - (KPG - 1) - first;   // plain: st * kKeys <= lim
  const int plain = min(nst, lim >= 0 ? lim / kKeys + 1 : 0);
  int st = 0;
  for (; st < plain; ++st) {
    next_stage(st);
#pragma unroll
    for (int half = 0; half < KPG / 32; ++half) {
      f32x4 s[kRB][2];
      products(s, ring + (st % kStages) * STAGE, kgrp + half);
      plain_block(s);
    }
  }
  for (; st < nst; ++st) {
    next_stage(st);
#pragma unroll
    for (int half = 0; half < KPG / 32; ++half) {
      const int kk0 = st * kKeys + first + half * 32;
      if (kk0 > wlast) break;   // (wave-uniform)
      f32x4 s[kRB][2];
      products(s, ring + (st % kStages) * STAGE, kgrp + half);
      edge_block(s, kk0);
    }
  }

  wait_vm<0>();   // (a workgroup with no live row has not waited for its first copies)

  // merge the four quads' states of every row (fixed order: xor 16, then xor 32), then the key groups' through LDS
  auto merge = [](float& m1, float& l1, float& e1, float m2, float l2, float e2) {
    const float M = fmaxf(m1, m2);
    if (M != -INFINITY) {
      rescale(m1, l1, e1, M);
      rescale(m2, l2, e2, M);
    }
    m1 = M;
    l1 += l2;
    e1 += e2;
  };
  if (KG > 1) barrier_lds();   // every wave is done with the ring
  float* st_lds = (float*)ring;   // [3][kRowsPerWg]: the second key group's states
  const int rl0 = (wave % kRowWaves) * kRowsPerWave;
#pragma unroll
  for (int rb = 0; rb < kRB; ++rb) {
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1)
      merge(m[rb], l[rb], e[rb], __shfl_xor(m[rb], off), __shfl_xor(l[rb], off), __shfl_xor(e[rb], off));
    if (kgrp == 1 && quad == 0) {
      const int rl = rl0 + rb * 16 + col;
      st_lds[rl] = m[rb];
      st_lds[kRowsPerWg + rl] = l[rb];
      st_lds[2 * kRowsPerWg + rl] = e[rb];
    }
  }
  if (KG > 1) barrier_lds();
  if (kgrp != 0 || quad != 0) return;
#pragma unroll
  for (int rb = 0; rb < kRB; ++rb) {
    const int rl = rl0 + rb * 16 + col;
    if (KG > 1) merge(m[rb], l[rb], e[rb], st_lds[rl], st_lds[kRowsPerWg + rl], st_lds[2 * kRowsPerWg + rl]);
    const int row = r0 + rl;
    if (row < a.N) {
      const bool live = row < nb && l[rb] > 0.f;
      if (a.lse) a.lse[qrow0 + row] = live ? (m[rb] + __log2f(l[rb])) * 0.69314718055994530942f : -INFINITY;
      if (a.entropy) a.entropy[qrow0 + row] = live ? 0.69314718055994530942f * (__log2f(l[rb]) - e[rb] / l[rb]) : 0.f;
    }
  }
}

// Mean of the prompt rows' entropies: sum over [B, Hq, N] (rows past n_b hold 0) / (Hq * sum_b n_b), fp64, in a
// fixed order (each thread a fixed stride of 16-byte vectors and the single entries at unaligned ends, then a tree
// over the threads).  One workgroup, bound by memory latency: 8 vectors a thread in flight (a load at a time took
// 26 us for 32 heads x 3136 rows; this form 6.4 us,
// 6.9 right after the statistics).
__global__ __launch_bounds__(1024) void prefill_entropy_mean_kernel(int B, int Hq, int N, const float* entropy,
                                                                    const int32_t* prompt_len, float* ae) {
  constexpr int U = 8;
  __shared__ double part[1024];
  const long long total = (long long)B * Hq * N;
  const int tid = threadIdx.x;
  const long long lead = (long long)((16 - ((uintptr_t)entropy & 15)) & 15) / 4;
  const long long head = lead < total ? lead : total, nv = (total - head) / 4;
  const f32x4* vec = (const f32x4*)(entropy + head);
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  for (long long i0 = tid; i0 < nv; i0 += U * 1024) {
    f32x4 x[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      x[k] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (i0 + k * 1024 < nv) x[k] = vec[i0 + k * 1024];
    }
    // (all of them in flight together: without this the loads move behind the branches below, one latency each)
    asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7]));
    static_assert(U == 8, "every vector is named");
#pragma unroll
    for (int k = 0; k < U; ++k) {
      // (a branch, so that a wave whose vectors are past the end skips the conversions: 8 heads x 300 rows 4.1 -> 3.6 us)
      if (i0 + k * 1024 >= nv) break;
      s0 += (double)x[k][0];
      s1 += (double)x[k][1];
      s2 += (double)x[k][2];
      s3 += (double)x[k][3];
    }
  }
  double s = (s0 + s1) + (s2 + s3);
  if (tid < head) s += (double)entropy[tid];
  if (head + 4 * nv + tid < total) s += (double)entropy[head + 4 * nv + tid];
  part[tid] = s;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if (tid < w) part[tid] += part[tid + w];
    __syncthreads();
  }
  if (tid == 0) {
    long long rows = 0;
    for (int b = 0; b < B; ++b) {
      const int nb = prompt_len[b];
      rows += nb < 0 ? 0 : (nb > N ? N : nb);
    }
    *ae = rows > 0 ? (float)(part[0] / ((double)Hq * (double)rows)) : 0.f;
  }
}

}  // namespace

template <int D, int KG>
hipError_t launch_stats(const PrefillArgs& a, hipStream_t stream) {
  constexpr size_t lds = (size_t)kStages * kKeys * D * 2;
  constexpr int rows = kRowsPerWgMax / KG;
  static bool configured = false;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)prefill_stats_kernel<D, KG>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const long long grid = (long long)a.B * a.Hq * ((a.N + rows - 1) / rows);
  hipLaunchKernelGGL((prefill_stats_kernel<D, KG>), dim3((unsigned)grid), dim3(64 * kWaves), lds, stream, a);
  return hipGetLastError();
}

// 256 rows a workgroup where that leaves four workgroups a compute unit (two, of one block each) and pads the rows by
// no more than a tenth beyond 128-row blocks: the two key groups' uneven ends and their merge cost more there than the
// shorter workgroups gain.  128 and 256 rows (us, head_dim 128): 16 x 40 heads x 500 rows 61, 52; x 256 27.3, 24.6;
// 8 x 40 x 1024 77, 70; 4 x 32 x 2000 105, 88; 32 x 32 x 200 35, 28; but 32 x 3136 61, 67; 2 x 32 x 3136 107, 110;
// 16 x 40 x 384 41, 44.  A prompt of at most 64 rows is one stage: 6.5, 6.0.
template <int D>
hipError_t launch_stats_rows(const PrefillArgs& a, hipStream_t stream) {
  const long long half = (a.N + kRowsPerWgMax / 2 - 1) / (kRowsPerWgMax / 2), whole = (half + 1) / 2;
  const long long grid = (long long)a.B * a.Hq * whole;
  if (a.N <= kKeys || (20 * whole <= 11 * half && grid >= (whole == 1 ? 2LL : 4LL) * a.cus))
    return launch_stats<D, 1>(a, stream);
  return launch_stats<D, 2>(a, stream);
}

hipError_t launch_prefill_stats(const PrefillArgs& a, hipStream_t stream) {
  if (a.B * (long long)a.Hq == 0) return hipSuccess;
  if (a.D == 128) return launch_stats_rows<128>(a, stream);
  if (a.D == 64) return launch_stats_rows<64>(a, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_prefill_entropy_mean(int B, int Hq, int N, const float* entropy, const int32_t* prompt_len, float* ae,
                                       hipStream_t stream) {
  hipLaunchKernelGGL(prefill_entropy_mean_kernel, dim3(1), dim3(1024), 0, stream, B, Hq, N, entropy, prompt_len, ae);
  return hipGetLastError();
}

}  // namespace dreams
