// What a workgroup of the generic attention kernel and of the few-row generic LM head does: each has a kernel of its own, and a
// whole verification step of a small call runs both in one launch.
#pragma once
#include "common.hpp"

namespace aurora {

constexpr int kGenThreads = 256;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// Sixteen bytes of a stored row, widened to fp32: 4 float32, 8 bfloat16 or 16 E4M3 elements.
template <typename TKV> struct Vec16 { static constexpr int n = 16 / (int)sizeof(TKV); float x[16 / sizeof(TKV)]; };
template <typename TKV>
__device__ __forceinline__ Vec16<TKV> load16(const TKV* p) {
  typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_t;
  const u32x4_t raw = *(const u32x4_t*)p;
  TKV e[Vec16<TKV>::n];
  __builtin_memcpy(e, &raw, 16);
  Vec16<TKV> r;
#pragma unroll
  for (int i = 0; i < Vec16<TKV>::n; ++i) r.x[i] = to_f32<TKV>(e[i]);
  return r;
}

// TKV = T, or e4m3_t with k_scale / v_scale [Hkv]: the scale of the KV head multiplies the scores and
// the weighted value sum (both are linear in it).  kD: head_dim.  kWhole: every request fits one split, out (and lse_out,
// or NULL) are written here.
template <typename T, typename TKV, int kD, bool kWhole>
__device__ __forceinline__ void attn_generic_part(
    int split, int hq, int bn, const T* __restrict__ q, const TKV* __restrict__ kp, const TKV* __restrict__ vp,
    const float* __restrict__ k_scale, const float* __restrict__ v_scale,
    const int32_t* __restrict__ block_table, const int32_t* __restrict__ seq_lens,
    const int32_t* __restrict__ parents, float* __restrict__ part_o, float* __restrict__ part_ml, T* __restrict__ out,
    float* __restrict__ lse_out, int Nq, int Hq, int Hkv, int page, int max_pages, int split_len, int max_splits, float scale) {
  constexpr int kWaves = kGenThreads / kWave;
  __shared__ __attribute__((aligned(16))) float q_s[kD];
  extern __shared__ __attribute__((aligned(16))) float sc[];  // split_len scores, then as many row numbers in the pools
  __shared__ float s_max[kWaves], s_sum[kWaves];
  __shared__ __attribute__((aligned(16))) f32x4_t s_o[kGenThreads];
  __shared__ unsigned long long anc_s;
  // (a pool has fewer than 2^32 rows of at least 64 bytes: K and V together would exceed the device's memory)
  uint32_t* rows = (uint32_t*)(sc + split_len);

  const int b = bn / Nq, n = bn % Nq;
  const int tid = threadIdx.x, lane = tid % kWave, wv = tid / kWave;
  const int L = seq_lens[b];
  const int start = split * split_len;
  const size_t orow = (size_t)bn * Hq + hq;
  if (start >= L) {
    if (kWhole) {  // an empty request: zeros, as the merge of no partial gives
      for (int d = tid; d < kD; d += kGenThreads) out[orow * kD + d] = from_f32<T>(0.f);
      if (lse_out && tid == 0) lse_out[orow] = -INFINITY;
    }
    return;
  }
  const int end = min(L, start + split_len);
  const int prefix = L - Nq;
  const int hk = hq / (Hq / Hkv);
  if (k_scale) scale *= k_scale[hk];
  const float vs = v_scale ? v_scale[hk] : 1.f;

  if (tid == 0) {
    unsigned long long m = 0;
    if (parents) {
      for (int a = n, hops = 0; a >= 0 && hops <= Nq; a = parents[b * Nq + a], ++hops) m |= 1ull << a;
    } else {
      m = n == 63 ? ~0ull : ((1ull << (n + 1)) - 1);
    }
    anc_s = m;
  }
  for (int d = tid; d < kD; d += kGenThreads) q_s[d] = to_f32<T>(q[orow * kD + d]);
  __syncthreads();
  const unsigned long long anc = anc_s;

  float lmax = -INFINITY;
  for (int j = start + tid; j < end; j += kGenThreads) {
    const bool seen = j < prefix || ((anc >> (j - prefix)) & 1ull);
    float s = -INFINITY;
    if (seen) {
      const int pj = j / page;
      const int pg = block_table[(size_t)b * max_pages + pj];
      const uint32_t r = ((uint32_t)pg * Hkv + hk) * (uint32_t)page + (uint32_t)(j - pj * page);
      rows[j - start] = r;
      const TKV* kr = kp + (size_t)r * kD;
      constexpr int kV = Vec16<TKV>::n;
      f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < kD / kV; ++c) {
        const Vec16<TKV> k = load16(kr + c * kV);
#pragma unroll
        for (int e = 0; e < kV; e += 4) {
          const f32x4_t qv = *(const f32x4_t*)(q_s + c * kV + e);
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[i] = fmaf(qv[i], k.x[e + i], acc[i]);
        }
      }
      s = ((acc[0] + acc[1]) + (acc[2] + acc[3])) * scale;
    }
    sc[j - start] = s;
    lmax = fmaxf(lmax, s);
  }
  lmax = wave_max(lmax);
  if (lane == 0) s_max[wv] = lmax;
  __syncthreads();
  float m = s_max[0];
#pragma unroll
  for (int i = 1; i < kWaves; ++i) m = fmaxf(m, s_max[i]);
  float lsum = 0.f;
  for (int j = start + tid; j < end; j += kGenThreads) {
    const float s = sc[j - start];
    const float p = (s == -INFINITY) ? 0.f : __expf(s - m);
    sc[j - start] = p;
    lsum += p;
  }
  lsum = wave_sum(lsum);
  if (lane == 0) s_sum[wv] = lsum;
  __syncthreads();
  float l = s_sum[0];
#pragma unroll
  for (int i = 1; i < kWaves; ++i) l += s_sum[i];

  // weighted value sum: thread (d4, g) adds columns 4 d4 .. of the positions j == g (mod groups)
  constexpr int kD4 = kD / 4, kGroups = kGenThreads / kD4;
  const int d4 = tid % kD4, g = tid / kD4;
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int j = g; j < end - start; j += kGroups) {
    const float p = sc[j];
    if (p != 0.f) {
      const TKV* vr = vp + (size_t)rows[j] * kD + 4 * d4;
      TKV e[4];
      __builtin_memcpy(e, __builtin_assume_aligned(vr, 4 * sizeof(TKV)), 4 * sizeof(TKV));
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = fmaf(p, to_f32<TKV>(e[i]), acc[i]);
    }
  }
  s_o[tid] = acc;
  __syncthreads();
  if (g != 0) return;
#pragma unroll
  for (int gg = 1; gg < kGroups; ++gg) acc += s_o[gg * kD4 + d4];
  if constexpr (kWhole) {
#pragma unroll
    for (int i = 0; i < 4; ++i) out[orow * kD + 4 * d4 + i] = from_f32<T>(l > 0.f ? acc[i] * vs / l : 0.f);
    if (lse_out && tid == 0) lse_out[orow] = l > 0.f ? m + __logf(l) : -INFINITY;
  } else {
    const size_t pidx = orow * max_splits + split;
    *(f32x4_t*)(part_o + pidx * kD + 4 * d4) = acc * vs;
    if (tid == 0) {
      part_ml[pidx * 2 + 0] = m;
      part_ml[pidx * 2 + 1] = l;
    }
  }
}

// The same product for few token rows: 64 x 64 tiles would leave most of the chip idle (16 workgroups on 20 x 1024) and walk
// the hidden dimension in steps of 16 with two barriers each.  Here a workgroup takes 16 vocabulary rows x 32 token rows and
// 64 hidden elements per step, the next step's operands being loaded into registers (16 bytes a thread) while the present
// ones are multiplied out of LDS; a thread owns one vocabulary row and two token rows.  20 x 1024 x 256 in fp32: 25 -> 6 us.
constexpr int kSM = 32, kSN = 16, kSK = 64, kSPad = 4;
template <typename T>
__device__ __forceinline__ void lmhead_few_tile(int bx, int by, const T* __restrict__ hidden, const T* __restrict__ w,
                                                float* __restrict__ logits, int64_t M, int H, int V) {
  __shared__ __attribute__((aligned(16))) float As[kSM][kSK + kSPad];
  __shared__ __attribute__((aligned(16))) float Bs[kSN][kSK + kSPad];
  const int tid = threadIdx.x;
  const int v0 = bx * kSN;
  const int64_t m0 = (int64_t)by * kSM;
  // staging: thread (r, c) brings elements 4c .. of rows r, r + 16 of the token tile and of row r of the vocabulary tile
  const int r = tid >> 4, c = (tid & 15) * 4;
  const bool vec = (H & 3) == 0;
  auto fetch = [&](const T* p, bool ok, int k) -> f32x4_t {
    f32x4_t x = {0.f, 0.f, 0.f, 0.f};
    if (ok && vec) {  // rows start at multiples of four elements
      if (k < H) {
        T t[4];
        __builtin_memcpy(t, __builtin_assume_aligned(p + k, 4 * sizeof(T)), 4 * sizeof(T));
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = to_f32<T>(t[e]);
      }
    } else if (ok) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (k + e < H) x[e] = to_f32<T>(p[k + e]);
    }
    return x;
  };
  const int64_t ma = m0 + r, mb = m0 + r + 16;
  const T* pa = hidden + (ma < M ? ma : 0) * H;
  const T* pb = hidden + (mb < M ? mb : 0) * H;
  const T* pw = w + (int64_t)(v0 + r < V ? v0 + r : 0) * H;
  const int n = tid & 15, mm = tid >> 4;  // this thread's vocabulary row; token rows mm and mm + 16
  f32x4_t acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
  f32x4_t xa = fetch(pa, ma < M, c), xb = fetch(pb, mb < M, c), xw = fetch(pw, v0 + r < V, c);
  for (int k0 = 0; k0 < H; k0 += kSK) {
    *(f32x4_t*)&As[r][c] = xa;
    *(f32x4_t*)&As[r + 16][c] = xb;
    *(f32x4_t*)&Bs[r][c] = xw;
    __syncthreads();
    if (k0 + kSK < H) {
      xa = fetch(pa, ma < M, k0 + kSK + c);
      xb = fetch(pb, mb < M, k0 + kSK + c);
      xw = fetch(pw, v0 + r < V, k0 + kSK + c);
    }
#pragma unroll
    for (int k = 0; k < kSK; k += 4) {
      const f32x4_t wv = *(const f32x4_t*)&Bs[n][k];
      const f32x4_t a0 = *(const f32x4_t*)&As[mm][k], a1 = *(const f32x4_t*)&As[mm + 16][k];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc0[e] = fmaf(a0[e], wv[e], acc0[e]);
        acc1[e] = fmaf(a1[e], wv[e], acc1[e]);
      }
    }
    __syncthreads();
  }
  const int v = v0 + n;
  if (v < V) {
    if (m0 + mm < M) logits[(m0 + mm) * V + v] = (acc0[0] + acc0[1]) + (acc0[2] + acc0[3]);
    if (m0 + mm + 16 < M) logits[(m0 + mm + 16) * V + v] = (acc1[0] + acc1[1]) + (acc1[2] + acc1[3]);
  }
}

}  // namespace aurora
