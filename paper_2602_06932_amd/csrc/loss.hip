// Drafter training loss on a batch of trace rows (paper section 3.3, eq. 3):
//
//   L = mean_{accepted rows} KL(p_target || p_draft) + lambda_discard * mean_{discarded rows} KL(p_target || p_draft)
//
// with its gradient with respect to the drafter's logits, w_m (p_draft - p_target).  p_target of a row is
// the softmax over the target logits kept for it (the K largest, appendix A.2; on discarded rows only the
// first discard_top_k of them - the paper's top-k filtering of discarded tokens), p_draft the softmax of
// the drafter's logits over its whole vocabulary.  Row classes are the trajectory codes of the trace
// record (appendix A.1): 1 accepted, 2 discarded, 0 unused.
//
// One workgroup per row and a fixed-order fp64 reduction of the row values; many rows have their classes counted by a
// kernel of its own first, of few every row's workgroup counts them by itself.
#include "launch.hpp"

namespace aurora {

constexpr int kLossThreads = 1024;
constexpr int kLossWaves = kLossThreads / kWave;

template <int kWaves = kLossWaves>
__device__ __forceinline__ float block_max(float v, float* s_red) {
  v = wave_max(v);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  __syncthreads();  // s_red may still be read from the previous reduction
  if (lane == 0) s_red[wv] = v;
  __syncthreads();
  float r = s_red[0];
#pragma unroll
  for (int i = 1; i < kWaves; ++i) r = fmaxf(r, s_red[i]);
  return r;
}

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}
template <int kWaves = kLossWaves, typename T>
__device__ __forceinline__ T block_sum(T v, T* s_red) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) s_red[wv] = v;
  __syncthreads();
  T r = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) r += s_red[i];  // fixed order
  return r;
}

__global__ __launch_bounds__(kLossThreads) void loss_count_kernel(const int8_t* __restrict__ traj, int M,
                                                                   float* __restrict__ loss_out) {
  __shared__ double s_red[kLossWaves];
  double na = 0.0, nd = 0.0;
  for (int m = threadIdx.x; m < M; m += kLossThreads) {
    const int c = traj[m];
    na += c == 1;
    nd += c == 2;
  }
  na = block_sum(na, s_red);
  nd = block_sum(nd, s_red);
  if (threadIdx.x == 0) {
    loss_out[3] = (float)na;
    loss_out[4] = (float)nd;
  }
}

// One workgroup per row.  kRounds > 0: a row of at most 4 kThreads kRounds values stays in registers: it is read once, each
// exponential is taken once, and the gradient is that exponential times w / sum.  At 128 registers a thread (512 threads, 16
// rounds) two rows share a compute unit, so one row's loads and stores overlap another's reductions.
// A row need not start at 16 bytes: the vectors start at its first aligned element, and the up to three elements before and
// after them are held by six threads.
// The kernel is bound by the row's bytes in and out, so every line of the gradient is written once and whole: w p_target is
// laid out in LDS, half a row at a time (the ids are distinct, a plain scatter; the first half while the row is on its way),
// and subtracted before the store.  Rewriting the kept tokens' entries in global memory afterwards found their lines
// partly evicted - 64 rows are in flight per 4 MB L2 - and cost 4 M partial writes (245 us at 4096 rows x 32000, 1024 kept).
// Loads return in order, so nothing between the row's loads and their use may wait for a load asked for after them: with the
// target side's loads behind the row's the same kernel takes 228 us, with them in front 207 us = 5.2 TB/s.  64 kept tokens,
// 2793 rows: 145 -> 140 us; 900 rows x 16001, which took three passes for want of alignment: 90 -> 38 us.
// Short rows are bound by the chain of reductions, so what counts is how many rows a compute unit holds, so up to
// 8192 values take four rounds - of 256 threads (68 registers, 16 KB of LDS: seven rows a unit) or of 512 (64 registers, 32 KB:
// four).  Against three rows of 256 threads and 32 rounds, and two of 512 and 16, grad included: 65536 rows x 40: 950 and 1291
// -> 328 us; 16384 x 512: 245 and 333 -> 93; 8192 x 4096, 1024 kept: 178 and 194 -> 80; 8192 x 8192: 210 and 202 -> 135.
// kRounds = 0 (rows longer than 32768 or shorter than 8, draft_logits and grad aligned differently): three passes over the row,
// the second and third from L2.
constexpr int kMaxKept = 1024;
constexpr int kScatRounds = 8;  // rounds per turn of the scatter, at most: 64 KB of LDS for 512 threads, two workgroups a unit
constexpr int kGridRows = 1 << 22;  // rows along the grid's first dimension: fewer than 2^32 threads; the rest along the second
// Rows are given to 256 threads up to here, four rounds in registers; then to 512, four rounds up to twice as much and sixteen
// beyond.
constexpr int kShortVals = 4096, kMidVals = 8192, kLongVals = 32768;
// Up to here a row's workgroup counts the classes itself (a few KB from L2 in place of a launch; short rows: as much as the rest
// of the row, so sooner not)
__host__ __device__ constexpr int count_rows(int threads) { return threads == 256 ? 2048 : 8192; }
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// whether the rows' workgroups count the classes themselves (their sums are the same whoever forms them)
__host__ __device__ inline bool counts_classes(const LossLaunch& P) {
  return P.grad && P.M <= count_rows(P.Vd <= kShortVals ? 256 : 512) && ((uintptr_t)P.traj & 3) == 0;
}

template <int kRowThreads, int kRounds>
__global__ __launch_bounds__(kRowThreads, kRounds == 0 ? 1 : kRounds > 4 ? 4 : kRowThreads == 256 ? 6 : 8) void loss_rows_kernel(LossLaunch P) {
  constexpr bool kInRegs = kRounds > 0;
  constexpr int kRowRounds = kInRegs ? kRounds : 1, kScat = kRowRounds < kScatRounds ? kRowRounds : kScatRounds;
  constexpr int kScatVals = kScat * kRowThreads * 4;
  constexpr int kRowWaves = kRowThreads / kWave, kRowKept = kMaxKept / kRowThreads;
  constexpr int kCountWords = count_rows(kRowThreads) / 4 / kRowThreads;
  __shared__ float s_redf[kRowWaves];
  __shared__ double s_redd[kRowWaves];
  const int tid = threadIdx.x;
  const long long row = (long long)blockIdx.y * kGridRows + blockIdx.x;
  if (row >= P.M) return;  // the whole workgroup
  const int m = (int)row;
  const int Vd = P.Vd, K = P.K;
  const float* z = P.draft_logits + (size_t)m * Vd;
  // elements before the first 16-byte boundary, vectors, and the first element after them (in registers only)
  const int h = kInRegs ? min((int)(((16 - ((uintptr_t)z & 15)) & 15) >> 2), Vd) : 0;
  const int n4 = (Vd - h) / 4, tail = h + 4 * n4;

  // What the target side needs is asked for first, the row behind it: loads return in order, so the target distribution, the
  // class counts and the weight are worked out while the row is on its way.
  const int cls = P.traj[m];
  // rows of the two classes, counted here if they are few: four codes a load
  const bool count = counts_classes(P);
  uint32_t c4[kCountWords];
#pragma unroll
  for (int e = 0; e < kCountWords; ++e) {
    const int i = tid + e * kRowThreads;
    c4[e] = 0u;
    if (count && 4 * i < P.M) {
      if (4 * i + 3 < P.M) {
        c4[e] = ((const uint32_t*)P.traj)[i];
      } else {
        for (int k = 4 * i; k < P.M; ++k) c4[e] |= (uint32_t)(uint8_t)P.traj[k] << (8 * (k & 3));
      }
    }
  }
  // thread t holds kept entries t, t + kRowThreads, ... (past the list: its last entry, sorted out below - a load under a condition
  // would be waited for at once)
  int id[kRowKept];
  uint16_t lt_bits[kRowKept];
#pragma unroll
  for (int e = 0; e < kRowKept; ++e) {
    const size_t at = (size_t)m * K + min(tid + e * kRowThreads, K - 1);
    id[e] = P.topk_ids[at];
    lt_bits[e] = P.topk_logits[at];
  }
  float n_acc = 0.f, n_disc = 0.f;
  if (P.grad && !count) {
    n_acc = P.loss_out[3];
    n_disc = P.loss_out[4];
  }
  asm volatile("" ::: "memory");

  f32x4_t r[kInRegs ? kRowRounds : 1];
  int edge = -1;  // the element outside the vectors that this thread holds
  float r_edge = -INFINITY;
  if constexpr (kInRegs) {
#pragma unroll
    for (int j = 0; j < kRowRounds; ++j) {
      const int i = tid + j * kRowThreads;
      r[j] = *((const f32x4_t*)(z + h) + min(i, n4 - 1));  // (past the end: re-read, and masked below)
    }
    if (tid < 3 && tid < h) edge = tid;
    if (tid >= 4 && tid < 7 && tail + tid - 4 < Vd) edge = tail + tid - 4;
    if (edge >= 0) r_edge = z[edge];
  }
  int na = 0, nd = 0;
#pragma unroll
  for (int e = 0; e < kCountWords; ++e)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int c = (int8_t)(c4[e] >> (8 * k));
      na += c == 1;
      nd += c == 2;
    }

  // ---- the row's target distribution ---------------------------------------------------------------------
  const int k_eff = (cls == 2 && P.discard_k > 0) ? min(P.discard_k, K) : K;
  float lt[kRowKept], zt_at[kRowKept];
  bool kept[kRowKept];
  float tmax = -INFINITY;
#pragma unroll
  for (int e = 0; e < kRowKept; ++e) {
    lt[e] = __uint_as_float((uint32_t)lt_bits[e] << 16);
    kept[e] = tid + e * kRowThreads < k_eff && id[e] >= 0 && id[e] < Vd && lt[e] > -INFINITY;
    tmax = fmaxf(tmax, kept[e] ? lt[e] : -INFINITY);
  }
#pragma unroll
  for (int e = 0; e < kRowKept; ++e) zt_at[e] = z[kept[e] ? id[e] : 0];  // the drafter's logit of the kept token
  tmax = block_max<kRowWaves>(tmax, s_redf);
  const bool any = tmax > -INFINITY;  // a row without a kept target logit contributes nothing
  double tsum = 0.0;
#pragma unroll
  for (int e = 0; e < kRowKept; ++e) tsum += kept[e] ? (double)__expf(lt[e] - tmax) : 0.0;
  tsum = block_sum<kRowWaves>(tsum, s_redd);
  const double lse_t = (double)tmax + log(tsum);

  float pt[kRowKept];
#pragma unroll
  for (int e = 0; e < kRowKept; ++e) pt[e] = kept[e] ? __expf((float)((double)lt[e] - lse_t)) : 0.f;

  // ---- the row's weight, and its share of w p_target laid out in LDS for the first turn of the gradient below ------------
  float w = 0.f;
  if (P.grad) {
    if (count) {  // both in one sum of whole numbers
      const int both = (int)block_sum<kRowWaves>((double)(na + (nd << 14)), s_redd);
      n_acc = (float)(both & ((1 << 14) - 1));
      n_disc = (float)(both >> 14);
    }
    if (any && cls == 1) w = 1.f / n_acc;
    if (any && cls == 2) w = P.lambda / n_disc;
  }
  constexpr int kLdsVals = kInRegs ? kScatVals : 4;
  __shared__ __attribute__((aligned(16))) float s_pt[kLdsVals];
  __shared__ float s_edge[8];
  auto scatter = [&](int first) {  // entries first .. of the vectors (distinct ids: a plain scatter)
#pragma unroll
    for (int e = 0; e < kRowKept; ++e)
      if (kept[e] && id[e] >= first && id[e] < min(first + kScatVals, tail)) s_pt[id[e] - first] = w * pt[e];
  };
  if constexpr (kInRegs) {
    if (P.grad) {
      const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < kScat; ++j) *(f32x4_t*)(s_pt + 4 * (tid + j * kRowThreads)) = zero;
      if (tid < 8) s_edge[tid] = 0.f;
      __syncthreads();
#pragma unroll
      for (int e = 0; e < kRowKept; ++e)
        if (kept[e]) {
          if (id[e] < h) s_edge[id[e]] = w * pt[e];
          if (id[e] >= tail) s_edge[4 + id[e] - tail] = w * pt[e];
        }
      scatter(h);  // the reductions below put barriers between this and its readers
    }
  }

  // ---- the drafter's logsumexp over its whole vocabulary ---------------------------------------------------
  const bool vec_ok = (Vd & 3) == 0 && ((uintptr_t)P.draft_logits & 15) == 0;
  float zmax = -INFINITY;
  double zsum = 0.0;
  if constexpr (kInRegs) {
    const f32x4_t ninf = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int j = 0; j < kRowRounds; ++j)
      if (tid + j * kRowThreads >= n4) r[j] = ninf;
#pragma unroll
    for (int j = 0; j < kRowRounds; ++j) zmax = fmaxf(zmax, fmaxf(fmaxf(r[j][0], r[j][1]), fmaxf(r[j][2], r[j][3])));
    zmax = fmaxf(zmax, r_edge);
    zmax = block_max<kRowWaves>(zmax, s_redf);
#pragma unroll
    for (int j = 0; j < kRowRounds; ++j) {
#pragma unroll
      for (int e = 0; e < 4; ++e) r[j][e] = __expf(r[j][e] - zmax);  // exp(-inf) = 0 past the end of the row
      zsum += ((double)r[j][0] + (double)r[j][1]) + ((double)r[j][2] + (double)r[j][3]);
      __builtin_amdgcn_sched_barrier(0);
    }
    r_edge = edge >= 0 ? __expf(r_edge - zmax) : 0.f;
    zsum += (double)r_edge;
  } else {
    if (vec_ok) {
      const float4* z4 = (const float4*)z;
      for (int i = tid; i < n4; i += kRowThreads) {
        const float4 x = z4[i];
        zmax = fmaxf(zmax, fmaxf(fmaxf(x.x, x.y), fmaxf(x.z, x.w)));
      }
    } else {
      for (int v = tid; v < Vd; v += kRowThreads) zmax = fmaxf(zmax, z[v]);
    }
    zmax = block_max<kRowWaves>(zmax, s_redf);
    if (vec_ok) {
      const float4* z4 = (const float4*)z;
      for (int i = tid; i < n4; i += kRowThreads) {
        const float4 x = z4[i];
        zsum += (double)__expf(x.x - zmax) + (double)__expf(x.y - zmax) + (double)__expf(x.z - zmax) +
                (double)__expf(x.w - zmax);
      }
    } else {
      for (int v = tid; v < Vd; v += kRowThreads) zsum += (double)__expf(z[v] - zmax);
    }
  }
  zsum = block_sum<kRowWaves>(zsum, s_redd);
  const double lse_d = (double)zmax + log(zsum);
  const float lse_df = (float)lse_d;

  // ---- KL(p_target || p_draft) of the row --------------------------------------------------------------------
  double term = 0.0;
#pragma unroll
  for (int e = 0; e < kRowKept; ++e)
    term += kept[e] ? (double)pt[e] * ((double)lt[e] - lse_t - ((double)zt_at[e] - lse_d)) : 0.0;
  const double kl = block_sum<kRowWaves>(term, s_redd);
  if (tid == 0) P.row_kl[m] = any ? (float)kl : 0.f;

  // ---- gradient: w (p_draft - p_target) ------------------------------------------------------------------------
  if (!P.grad) return;
  float* g = P.grad + (size_t)m * Vd;
  if constexpr (kInRegs) {
    const float scale = w * (float)(1.0 / zsum);
    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j0 = 0; j0 < kRowRounds; j0 += kScat) {
      if (j0 * kRowThreads >= n4) break;  // uniform
      if (j0 > 0) {
        __syncthreads();  // the turn before has been read and cleared
        scatter(h + 4 * j0 * kRowThreads);
        __syncthreads();
      }
#pragma unroll
      for (int j = 0; j < kScat; ++j) {
        const int i = tid + (j0 + j) * kRowThreads;
        f32x4_t* at = (f32x4_t*)(s_pt + 4 * (tid + j * kRowThreads));
        const f32x4_t o = r[j0 + j] * scale - *at;
        if (j0 + kScat < kRowRounds) *at = zero;  // for the next turn; nobody else reads it
        if (i < n4) *((f32x4_t*)(g + h) + i) = o;
        __builtin_amdgcn_sched_barrier(0);  // one round at a time: nothing but r[] may take registers here
      }
    }
    if (edge >= 0) g[edge] = r_edge * scale - s_edge[tid];
    return;
  } else {
    const bool gvec = vec_ok && ((uintptr_t)P.grad & 15) == 0;
    if (gvec) {
      const float4* z4 = (const float4*)z;
      float4* g4 = (float4*)g;
      for (int i = tid; i < n4; i += kRowThreads) {
        const float4 x = z4[i];
        float4 o;
        o.x = w * __expf(x.x - lse_df);
        o.y = w * __expf(x.y - lse_df);
        o.z = w * __expf(x.z - lse_df);
        o.w = w * __expf(x.w - lse_df);
        g4[i] = o;
      }
    } else {
      for (int v = tid; v < Vd; v += kRowThreads) g[v] = w * __expf(z[v] - lse_df);
    }
  }
  __syncthreads();  // the kept tokens' entries are rewritten by other threads than those that wrote them above
#pragma unroll
  for (int e = 0; e < kRowKept; ++e)
    if (kept[e]) g[id[e]] = w * (__expf(zt_at[e] - lse_df) - pt[e]);
}

__global__ __launch_bounds__(kLossThreads) void loss_reduce_kernel(const float* __restrict__ row_kl,
                                                                    const int8_t* __restrict__ traj, int M, float lambda,
                                                                    float* __restrict__ loss_out) {
  __shared__ double s_red[kLossWaves];
  __shared__ unsigned long long s_cnt[kLossWaves];
  double sa = 0.0, sd = 0.0;
  unsigned long long both = 0;  // accepted rows below, discarded rows from bit 32 on (M < 2^31: neither reaches the other)
  for (int m = threadIdx.x; m < M; m += kLossThreads) {
    const int c = traj[m];
    const double x = (double)row_kl[m];
    if (c == 1) { sa += x; both += 1ull; }
    if (c == 2) { sd += x; both += 1ull << 32; }
  }
  sa = block_sum(sa, s_red);
  sd = block_sum(sd, s_red);
  both = block_sum(both, s_cnt);
  if (threadIdx.x == 0) {
    const double na = (double)(both & 0xffffffffull), nd = (double)(both >> 32);
    loss_out[3] = (float)na;
    loss_out[4] = (float)nd;
    const double ma = na > 0 ? sa / na : 0.0, md = nd > 0 ? sd / nd : 0.0;
    loss_out[0] = (float)(ma + (double)lambda * md);
    loss_out[1] = (float)ma;
    loss_out[2] = (float)md;
  }
}

int loss_max_k() { return kMaxKept; }

hipError_t launch_draft_loss(const LossLaunch& P, hipStream_t st) {
  hipError_t e;
  if (P.grad && !counts_classes(P)) {
    hipLaunchKernelGGL(loss_count_kernel, dim3(1), dim3(kLossThreads), 0, st, P.traj, P.M, P.loss_out);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (P.M > 0) {
    // rows and gradient rows have to start at the same place within 16 bytes
    const bool in_regs = P.Vd >= 8 && P.Vd <= kLongVals && (!P.grad || (((uintptr_t)P.grad ^ (uintptr_t)P.draft_logits) & 15) == 0);
    const dim3 grid(P.M < kGridRows ? P.M : kGridRows, (P.M - 1) / kGridRows + 1);
#define AURORA_LOSS_ROWS(T, R) hipLaunchKernelGGL((loss_rows_kernel<T, R>), grid, dim3(T), 0, st, P)
    if (P.Vd <= kShortVals) {
      if (in_regs) AURORA_LOSS_ROWS(256, 4); else AURORA_LOSS_ROWS(256, 0);
    } else {
      if (!in_regs) AURORA_LOSS_ROWS(512, 0);
      else if (P.Vd <= kMidVals) AURORA_LOSS_ROWS(512, 4);
      else AURORA_LOSS_ROWS(512, 16);
    }
#undef AURORA_LOSS_ROWS
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(kLossThreads), 0, st, P.row_kl, P.traj, P.M, P.lambda, P.loss_out);
  return hipGetLastError();
}

}  // namespace aurora
