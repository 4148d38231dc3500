// Tree-masked verification attention, fp32 inputs (the small fp32 workload: latency and launches, plain VALU).
//
// A workgroup of 16 waves owns R rows (1, 2 or 4) of one KV head and all of that head's keys.  A key's K (or V)
// row is held by D/4 neighbouring lanes, 16 bytes each, so a wave reads 64 / (D/4) whole rows per load, in full
// cache lines; U such groups of keys are in flight per wave and the 16 waves cover 16 U groups, so that 640 keys
// take three rounds of memory latency.  A score is four products per lane and a sum over the key's lanes
// (rotations within 16 lanes, every lane ends with it); each lane then owns 4 columns of the row's output.
// Every lane group keeps its own online softmax (running max, running sum, accumulator) in fp32; the states are
// merged within the wave, then across the waves in wave order through LDS, so results are reproducible.  What
// bounds it is the latency of the launch and of the first reads, and with many rows the reads of the keys by one
// compute unit: R rows share them.  A thread per key, each lane reading its key's rows alone (64 cache lines a
// load), took 20.9 us at 4 heads x 16 nodes x 640 keys and 231 us at 1600 rows x 1300 keys; this form takes 6.4 and
// 47 us.  Within a pass the keys are summed among themselves before the state takes them: the error against 64 bits
// is 1.05e-7 at the first shape (1.2e-7 before).
//
// With an entropy output, each state also carries e = sum 2^(x-m) (x-m) (scores x in log2 units), from which the
// row's attention entropy follows as ln2 * (log2 l - e/l); re-referencing a state to M with weight w = 2^(m-M)
// turns e into w (e + (m-M) l).
#include "kernels.h"

#include <math.h>
#include <type_traits>

namespace dreams {
namespace {

constexpr float kLn2 = 0.69314718055994530942f;
constexpr int kF32Waves = 16;

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float ent_term(float w, float e, float m, float M, float l) {
  return w == 0.f ? 0.f : w * fmaf(m - M, l, e);
}

// sum over the 16 lanes of a row of lanes, or over 32 neighbouring lanes; every lane gets the same bits (each
// step adds the same two values in both lanes of a pair)
template <int CTRL>
__device__ __forceinline__ float add_rotated(float x) {
  const int y = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true);
  return x + __builtin_bit_cast(float, y);
}
template <int LANES>
__device__ __forceinline__ float sum_lanes(float x) {
  x = add_rotated<0x128>(x);   // row_ror:8, 4, 2, 1
  x = add_rotated<0x124>(x);
  x = add_rotated<0x122>(x);
  x = add_rotated<0x121>(x);
  if constexpr (LANES == 32) x += __shfl_xor(x, 16);
  return x;
}

template <int D, int R>
__global__ __launch_bounds__(64 * kF32Waves) void tree_attn_f32_kernel(AttnArgs a) {
  constexpr int NW = kF32Waves;
  constexpr int LPK = D / 4;          // lanes per key
  constexpr int KPI = 64 / LPK;       // keys a wave reads per load
  constexpr int U = 4;                // such groups of keys per pass
  __shared__ int par_lds[kMaxNodes];
  __shared__ uint64_t anc_lds[R][2];
  __shared__ float st_mle[NW][R][3];
  __shared__ float st_acc[NW][R][D];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane % LPK, kg = lane / LPK;   // this lane's 16-byte piece of a row, and its key of a group
  const int T = a.T, rows_u = a.G * T;
  // workgroup n takes unit n % units, so that the workgroups of one KV head sit on as few XCDs as the unit count
  // allows (consecutive ids go round-robin over the 8) and share its keys in their L2
  const int u = (int)(blockIdx.x % (unsigned)a.units), r0 = (int)(blockIdx.x / (unsigned)a.units) * R;
  const int b = u / a.Hkv;
  int L = a.kv_len[b];
  L = L < 0 ? 0 : (L > a.S_cap - T ? a.S_cap - T : L);
  const size_t row0 = (size_t)u * rows_u;   // row 0 of this KV head's query rows
  const float* kb = (const float*)a.k + (size_t)u * a.S_cap * D + 4 * c;
  const float* vb = (const float*)a.v + (size_t)u * a.S_cap * D + 4 * c;

  f32x4 q[R], acc[R];
  float m[R], l[R], e[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    q[r] = *(const f32x4*)((const float*)a.q + (row0 + min(r0 + r, rows_u - 1)) * D + 4 * c);
    acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
    m[r] = -INFINITY;
    l[r] = 0.f;
    e[r] = 0.f;
  }
  // this wave's first tree keys (its group of them, clamped to the last node), read ahead of the prefix
  int jt = wave * KPI + kg;
  f32x4 kt = *(const f32x4*)(kb + (size_t)(L + min(jt, T - 1)) * D);
  f32x4 vt = *(const f32x4*)(vb + (size_t)(L + min(jt, T - 1)) * D);
  if (!a.mask && tid < T) par_lds[tid] = a.parent[(size_t)b * T + tid];
  __syncthreads();
  // the rows' ancestors-or-self: a walk in LDS by the last wave (or the mask rows); read after the prefix
  if (tid >= 64 * (NW - 1) && tid - 64 * (NW - 1) < R) {
    const int r = tid - 64 * (NW - 1);
    const int i = min(r0 + r, rows_u - 1) % T;
    uint64_t anc0 = 0, anc1 = 0;
    if (a.mask) {
      const int W = (T + 63) / 64;
      const uint64_t* mr = a.mask + ((size_t)b * T + i) * W;
      anc0 = mr[0];
      anc1 = W > 1 ? mr[1] : 0;
    } else {
      int j = i;
      for (int step = 0; step <= T && j >= 0; ++step) {
        if (j < 64) anc0 |= 1ull << j; else anc1 |= 1ull << (j - 64);
        const int p = par_lds[j];
        if (p >= j) break;
        j = p;
      }
    }
    anc_lds[r][0] = anc0;
    anc_lds[r][1] = anc1;
  }

  const bool ent = a.entropy != nullptr;
  // NK groups of keys into every row's state; masked: only the keys with see[r][t], whose values alone count
  auto update = [&](auto nk, auto masked, const f32x4* kk, const f32x4* vv, auto see) {
    constexpr int NK = decltype(nk)::value;
    constexpr bool MASKED = decltype(masked)::value;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float x[NK], mx = m[r];   // x: products (scaled inside the exponent, one rounding for both)
#pragma unroll
      for (int t = 0; t < NK; ++t) {
        float s = q[r][0] * kk[t][0];
        s = fmaf(q[r][1], kk[t][1], s);
        s = fmaf(q[r][2], kk[t][2], s);
        s = fmaf(q[r][3], kk[t][3], s);
        x[t] = sum_lanes<LPK>(s);
        if (!MASKED || see(r, t)) mx = fmaxf(mx, x[t] * a.scale_log2);
      }
      const float ref = mx == -INFINITY ? 0.f : mx;   // (nothing seen yet: every weight below is 2^-inf = 0)
      const float alpha = __builtin_amdgcn_exp2f(m[r] - ref);
      if (ent) e[r] = ent_term(l[r] == 0.f ? 0.f : alpha, e[r], m[r], ref, l[r]);
      // the pass's keys among themselves first, then onto the state: fewer roundings at the state's size
      float psum = 0.f, esum = 0.f;
      f32x4 pv = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < NK; ++t) {
        const float z = fmaf(x[t], a.scale_log2, -ref);
        const float p = MASKED && !see(r, t) ? 0.f : __builtin_amdgcn_exp2f(z);
        if (ent && p != 0.f) esum = fmaf(p, z, esum);
        psum += p;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float v = MASKED && !see(r, t) ? 0.f : vv[t][i];
          pv[i] = fmaf(p, v, pv[i]);
        }
      }
      if (ent) e[r] += esum;
      l[r] = fmaf(l[r], alpha, psum);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[r][i] = fmaf(acc[r][i], alpha, pv[i]);
      m[r] = mx;
    }
  };

  // ---- the prefix: passes of U groups of keys per wave
  for (int s0 = wave * (KPI * U); s0 < L; s0 += NW * KPI * U) {
    f32x4 kk[U], vv[U];
#pragma unroll
    for (int t = 0; t < U; ++t) kk[t] = *(const f32x4*)(kb + (size_t)min(s0 + t * KPI + kg, L - 1) * D);
#pragma unroll
    for (int t = 0; t < U; ++t) vv[t] = *(const f32x4*)(vb + (size_t)min(s0 + t * KPI + kg, L - 1) * D);
    if (s0 + KPI * U <= L)
      update(std::integral_constant<int, U>{}, std::false_type{}, kk, vv, [](int, int) { return true; });
    else
      update(std::integral_constant<int, U>{}, std::true_type{}, kk, vv,
             [&](int, int t) { return s0 + t * KPI + kg < L; });
  }
  // ---- the tree
  __syncthreads();
  for (int j0 = wave * KPI; j0 < T; j0 += NW * KPI) {
    const int j = j0 + kg;
    update(std::integral_constant<int, 1>{}, std::true_type{}, &kt, &vt, [&](int r, int) {
      return j < T && ((anc_lds[r][j >> 6] >> (j & 63)) & 1ull) != 0;
    });
    jt = min(j + NW * KPI, T - 1);
    if (j0 + NW * KPI < T) {
      kt = *(const f32x4*)(kb + (size_t)(L + jt) * D);
      vt = *(const f32x4*)(vb + (size_t)(L + jt) * D);
    }
  }

  // ---- the wave's lane groups, then the waves in wave order
#pragma unroll
  for (int r = 0; r < R; ++r) {
#pragma unroll
    for (int off = LPK; off < 64; off <<= 1) {
      const float mo = __shfl_xor(m[r], off), lo = __shfl_xor(l[r], off), eo = __shfl_xor(e[r], off);
      const float M = fmaxf(m[r], mo);
      const float w = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[r] - M);
      const float wo = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mo - M);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[r][i] = acc[r][i] * w + __shfl_xor(acc[r][i], off) * wo;
      if (ent) e[r] = ent_term(w, e[r], m[r], M, l[r]) + ent_term(wo, eo, mo, M, lo);
      l[r] = l[r] * w + lo * wo;
      m[r] = M;
    }
    if (kg == 0) *(f32x4*)&st_acc[wave][r][4 * c] = acc[r];
    if (lane == 0) {
      st_mle[wave][r][0] = m[r];
      st_mle[wave][r][1] = l[r];
      st_mle[wave][r][2] = e[r];
    }
  }
  __syncthreads();
  if (tid >= R * D) return;
  const int r = tid / D, d = tid % D;   // this thread's row and output column
  if (r0 + r >= rows_u) return;
  float M = st_mle[0][r][0];
#pragma unroll
  for (int w = 1; w < NW; ++w) M = fmaxf(M, st_mle[w][r][0]);
  float l4[4] = {}, e4[4] = {}, o4[4] = {};   // four chains, then their sums in pairs
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const float mw = st_mle[w][r][0], lw = st_mle[w][r][1], ew = st_mle[w][r][2];
    const float wt = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - M);
    if (ent) e4[w % 4] += ent_term(wt, ew, mw, M, lw);
    l4[w % 4] = fmaf(lw, wt, l4[w % 4]);
    o4[w % 4] = fmaf(st_acc[w][r][d], wt, o4[w % 4]);
  }
  const float lt = (l4[0] + l4[1]) + (l4[2] + l4[3]), et = (e4[0] + e4[1]) + (e4[2] + e4[3]);
  const float o = (o4[0] + o4[1]) + (o4[2] + o4[3]);
  const size_t row = row0 + r0 + r;
  ((float*)a.out)[row * D + d] = lt > 0.f ? o / lt : 0.f;
  if (a.lse && d == 0) a.lse[row] = lt > 0.f ? (M + log2f(lt)) * kLn2 : -INFINITY;
  if (ent && d == 0) a.entropy[row] = lt > 0.f ? kLn2 * (log2f(lt) - et / lt) : 0.f;
}

template <int D, int R>
hipError_t launch_f32(const AttnArgs& a, hipStream_t stream) {
  const unsigned grid = (unsigned)a.units * (unsigned)((a.G * a.T + R - 1) / R);
  hipLaunchKernelGGL((tree_attn_f32_kernel<D, R>), dim3(grid), dim3(64 * kF32Waves), 0, stream, a);
  return hipGetLastError();
}

// Rows per workgroup: 1 while that leaves at most one workgroup per compute unit, then 2, then 4.  A workgroup of
// 2 rows takes about 1.3 times, of 4 rows 2.2 times as long as one of 1 row, and a second round as long again
// (us at 1, 2 and 4 rows:
// 64 rows x 640 keys 6.4, 8.1, 13.8; 480 x 640 12.8, 9.2, 15.6; 1600 x 1300 65, 53, 49).  At the 128 registers a lane
// that 16 waves leave, 4 rows spill 11 (head_dim 64) or 13 (128) of them to scratch; those times include that.
template <int D>
hipError_t launch_f32_rows(const AttnArgs& a, hipStream_t stream) {
  const long long rows = (long long)a.units * a.G * a.T;
  if (rows <= a.cus) return launch_f32<D, 1>(a, stream);
  if (rows <= 2LL * a.cus) return launch_f32<D, 2>(a, stream);
  return launch_f32<D, 4>(a, stream);
}

}  // namespace

hipError_t launch_tree_attn_f32(const AttnArgs& a, hipStream_t stream) {
  if (a.D == 64) return launch_f32_rows<64>(a, stream);
  if (a.D == 128) return launch_f32_rows<128>(a, stream);
  return hipErrorInvalidValue;
}

}  // namespace dreams
