// Generic chunk attention (head_dim 64 or 128, any page size, fp32 or bf16 storage - or a KV cache of
// E4M3 codes with one scale per KV head - fp32 arithmetic).  It is the fp32 path of the library and the fallback for bf16 shapes the MFMA
// kernel does not cover.  One workgroup per (split, query head, request x node): scores for
// the split's visible KV positions, a block-wide max / sum, then the weighted value sum; a
// second kernel merges the splits (sections 3.1 and 3.2 of the paper define what is computed:
// the draft positions are verified in one pass, a tree under its ancestor mask).
//
// Small calls are what comes here, and they are bound by latency: a thread reads its token's whole key with 16-byte loads
// that are all in flight together, the page look-up is done once per token and kept for the value pass, reductions take two
// barriers, and where a request fits one split the workgroup writes the output itself.  4 requests x 5 positions x 8 heads
// over 256 tokens, fp32: 27 us + 4.8 us for the merge (one 4-byte load at a time, a division per element) -> 9.7 us.
#include "common.hpp"
#include "launch.hpp"

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
__global__ __launch_bounds__(kGenThreads) void attn_generic_partial(
    const T* __restrict__ q, const TKV* __restrict__ kp, const TKV* __restrict__ vp,
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

  const int split = blockIdx.x, hq = blockIdx.y, bn = blockIdx.z;
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

// Merge the per-split partials of one (request, node, query head): out = sum_s e^{m_s-M} O_s / sum_s e^{m_s-M} l_s.
template <typename T>
__global__ void attn_combine(const float* __restrict__ part_o, const float* __restrict__ part_ml,
                             const int32_t* __restrict__ seq_lens, T* __restrict__ out, int Nq, int Hq, int D,
                             int split_len, int max_splits, float* __restrict__ lse_out) {
  const size_t row = blockIdx.x;  // (b*Nq + n)*Hq + hq
  const int b = (int)(row / ((size_t)Nq * Hq));
  const int L = seq_lens[b];
  const int ns = min(max_splits, (L + split_len - 1) / split_len);
  const size_t base = row * max_splits;
  float M = -INFINITY;
  for (int s = 0; s < ns; ++s) M = fmaxf(M, part_ml[(base + s) * 2]);
  if (lse_out && threadIdx.x == 0) {
    float den = 0.f;
    for (int s = 0; s < ns; ++s) {
      const float ms = part_ml[(base + s) * 2];
      if (ms > -INFINITY) den = fmaf(__expf(ms - M), part_ml[(base + s) * 2 + 1], den);
    }
    lse_out[row] = den > 0.f ? M + __logf(den) : -INFINITY;
  }
  for (int d = threadIdx.x; d < D; d += blockDim.x) {
    float num = 0.f, den = 0.f;
    for (int s = 0; s < ns; ++s) {
      const float ms = part_ml[(base + s) * 2];
      const float w = (ms == -INFINITY) ? 0.f : __expf(ms - M);
      num = fmaf(w, part_o[(base + s) * D + d], num);
      den = fmaf(w, part_ml[(base + s) * 2 + 1], den);
    }
    out[row * D + d] = from_f32<T>(den > 0.f ? num / den : 0.f);
  }
}

template <typename T, typename TKV, int kD, bool kWhole>
static hipError_t launch_generic_k(const AttnLaunch& a, hipStream_t st) {
  dim3 grid(a.plan.max_splits, a.Hq, a.B * a.Nq);
  const size_t lds = (size_t)a.plan.split_len * (sizeof(float) + sizeof(uint32_t));
  hipLaunchKernelGGL((attn_generic_partial<T, TKV, kD, kWhole>), grid, dim3(kGenThreads), lds, st, (const T*)a.q,
                     (const TKV*)a.k, (const TKV*)a.v, a.kv_fp8 ? a.k_scale : nullptr, a.kv_fp8 ? a.v_scale : nullptr,
                     a.block_table, a.seq_lens, a.parents, a.part_o, a.part_ml, (T*)a.out, a.lse_out, a.Nq, a.Hq, a.Hkv,
                     a.page, a.max_pages, a.plan.split_len, a.plan.max_splits, a.scale);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  return kWhole ? hipSuccess : launch_attn_combine(a, st);
}

template <typename T, typename TKV>
static hipError_t launch_generic_t(const AttnLaunch& a, hipStream_t st) {
  const bool whole = a.plan.max_splits == 1;
  if (a.D == 64) return whole ? launch_generic_k<T, TKV, 64, true>(a, st) : launch_generic_k<T, TKV, 64, false>(a, st);
  return whole ? launch_generic_k<T, TKV, 128, true>(a, st) : launch_generic_k<T, TKV, 128, false>(a, st);
}

hipError_t launch_attn_combine(const AttnLaunch& a, hipStream_t st) {
  const unsigned rows = (unsigned)((size_t)a.B * a.Nq * a.Hq);
  if (a.bf16)
    hipLaunchKernelGGL(attn_combine<bf16_t>, dim3(rows), dim3(a.D <= 64 ? 64 : 128), 0, st, a.part_o, a.part_ml,
                       a.seq_lens, (bf16_t*)a.out, a.Nq, a.Hq, a.D, a.plan.split_len, a.plan.max_splits, a.lse_out);
  else
    hipLaunchKernelGGL(attn_combine<float>, dim3(rows), dim3(a.D <= 64 ? 64 : 128), 0, st, a.part_o, a.part_ml,
                       a.seq_lens, (float*)a.out, a.Nq, a.Hq, a.D, a.plan.split_len, a.plan.max_splits, a.lse_out);
  return hipGetLastError();
}

hipError_t launch_attn_generic(const AttnLaunch& a, hipStream_t st) {
  if (a.kv_fp8) return a.bf16 ? launch_generic_t<bf16_t, e4m3_t>(a, st) : launch_generic_t<float, e4m3_t>(a, st);
  return a.bf16 ? launch_generic_t<bf16_t, bf16_t>(a, st) : launch_generic_t<float, float>(a, st);
}

}  // namespace aurora
