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
#include "generic_tile.hpp"
#include "launch.hpp"

namespace aurora {

template <typename T, typename TKV, int kD, bool kWhole>
__global__ __launch_bounds__(kGenThreads) void attn_generic_partial(
    const T* __restrict__ q, const TKV* __restrict__ kp, const TKV* __restrict__ vp,
    const float* __restrict__ k_scale, const float* __restrict__ v_scale,
    const int32_t* __restrict__ block_table, const int32_t* __restrict__ seq_lens,
    const int32_t* __restrict__ parents, float* __restrict__ part_o, float* __restrict__ part_ml, T* __restrict__ out,
    float* __restrict__ lse_out, int Nq, int Hq, int Hkv, int page, int max_pages, int split_len, int max_splits, float scale) {
  attn_generic_part<T, TKV, kD, kWhole>(blockIdx.x, blockIdx.y, blockIdx.z, q, kp, vp, k_scale, v_scale, block_table, seq_lens,
                                        parents, part_o, part_ml, out, lse_out, Nq, Hq, Hkv, page, max_pages, split_len,
                                        max_splits, scale);
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
