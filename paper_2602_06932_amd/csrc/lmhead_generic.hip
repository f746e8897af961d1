// Generic LM-head projection (fp32 FMA, fp32 or bf16 storage) followed by per-tile softmax
// statistics.  It is the fp32 path of the library and the fallback for shapes the MFMA kernel
// does not cover.  logits[m, v] = sum_h hidden[m, h] * W[v, h]  (appendix A.1, eq. 4: l in R^{T x V}).
#include "generic_tile.hpp"
#include "launch.hpp"

namespace aurora {

constexpr int kTM = 64, kTN = 64, kTK = 16;

template <typename T>
__global__ __launch_bounds__(256) void lmhead_generic(const T* __restrict__ hidden, const T* __restrict__ w,
                                                      float* __restrict__ logits, int64_t M, int H, int V) {
  __shared__ float As[kTK][kTM + 4];
  __shared__ float Bs[kTK][kTN + 4];
  const int tid = threadIdx.x;
  const int tx = tid % 16, ty = tid / 16;
  const int64_t m0 = (int64_t)blockIdx.y * kTM;
  const int64_t v0 = (int64_t)blockIdx.x * kTN;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < H; k0 += kTK) {
    for (int i = tid; i < kTM * kTK; i += 256) {
      const int r = i / kTK, c = i % kTK;
      const int64_t m = m0 + r;
      const int k = k0 + c;
      As[c][r] = (m < M && k < H) ? to_f32<T>(hidden[m * H + k]) : 0.f;
      const int64_t v = v0 + r;
      Bs[c][r] = (v < V && k < H) ? to_f32<T>(w[v * H + k]) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < kTK; ++kk) {
      float a[4], bcol[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) bcol[j] = Bs[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], bcol[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t m = m0 + ty * 4 + i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t v = v0 + tx * 4 + j;
      if (v < V) logits[m * V + v] = acc[i][j];
    }
  }
}

template <typename T>
__global__ __launch_bounds__(256) void lmhead_generic_few(const T* __restrict__ hidden, const T* __restrict__ w,
                                                          float* __restrict__ logits, int64_t M, int H, int V) {
  lmhead_few_tile<T>(blockIdx.x, blockIdx.y, hidden, w, logits, M, H, V);
}

// Attention and LM head of a small call in one launch (float32, few token rows): workgroups [0, lm_x lm_y) take the head's
// tiles, the others a (request x node, query head, split) each; kWhole: one split holds every request.  Both are chains of memory round trips
// that leave most of the chip idle: side by side the longer one counts.  4 x 5 positions x 8 heads over 256 tokens and 20 x 1024
// logits: 9 + 6 us and a launch -> 10 us.
template <int kD, bool kWhole>
__global__ __launch_bounds__(kGenThreads) void verify_front_f32(AttnLaunch a, const float* __restrict__ hidden,
                                                                const float* __restrict__ w, float* __restrict__ logits,
                                                                int64_t M, int H, int V, int lm_x, int lm_y) {
  const int wg = blockIdx.x, n_lm = lm_x * lm_y;
  if (wg < n_lm) {
    lmhead_few_tile<float>(wg % lm_x, wg / lm_x, hidden, w, logits, M, H, V);
  } else {
    const int splits = kWhole ? 1 : a.plan.max_splits, split = (wg - n_lm) % splits, i = (wg - n_lm) / splits;
    attn_generic_part<float, float, kD, kWhole>(split, i % a.Hq, i / a.Hq, (const float*)a.q, (const float*)a.k, (const float*)a.v,
                                                nullptr, nullptr, a.block_table, a.seq_lens, a.parents, a.part_o, a.part_ml,
                                                (float*)a.out, nullptr, a.Nq, a.Hq, a.Hkv, a.page, a.max_pages, a.plan.split_len,
                                                splits, a.scale);
  }
}

// One workgroup per (vocab tile, row): max, arg-max (lowest index on ties) and
// sum exp((l - max) * inv_t) over the tile's columns.
__global__ __launch_bounds__(256) void row_tile_stats(const float* __restrict__ logits, float* __restrict__ pmax,
                                                      float* __restrict__ psum, int32_t* __restrict__ parg, int V,
                                                      int stat_tile, int n_tiles, float inv_t,
                                                      const float* __restrict__ temps, int Nq) {
  __shared__ float smax[4];
  __shared__ int sarg[4];
  __shared__ float ssum[4];
  const int tile = blockIdx.x;
  const int64_t row = blockIdx.y;
  const int tid = threadIdx.x, lane = tid % kWave, wv = tid / kWave;
  const int v0 = tile * stat_tile, v1 = min(V, v0 + stat_tile);
  const float* lr = logits + row * V;
  if (temps) {  // one temperature per request; 0 = greedy, statistics at T = 1
    const float T = temps[row / Nq];
    inv_t = T > 0.f ? 1.f / T : 1.f;
  }
  float mx = -INFINITY;
  int arg = 0x7fffffff;
  for (int v = v0 + tid; v < v1; v += 256) {
    const float x = lr[v];
    if (x > mx) { mx = x; arg = v; }  // ascending v per thread: first occurrence kept
  }
  // wave reduce (max, lowest index among equals)
  for (int o = 32; o > 0; o >>= 1) {
    const float om = __shfl_xor(mx, o, kWave);
    const int oa = __shfl_xor(arg, o, kWave);
    if (om > mx || (om == mx && oa < arg)) { mx = om; arg = oa; }
  }
  if (lane == 0) { smax[wv] = mx; sarg[wv] = arg; }
  __syncthreads();
  mx = smax[0]; arg = sarg[0];
  for (int i = 1; i < 4; ++i)
    if (smax[i] > mx || (smax[i] == mx && sarg[i] < arg)) { mx = smax[i]; arg = sarg[i]; }
  float s = 0.f;
  for (int v = v0 + tid; v < v1; v += 256) s += __expf((lr[v] - mx) * inv_t);
  s = wave_sum(s);
  if (lane == 0) ssum[wv] = s;
  __syncthreads();
  if (tid == 0) {
    pmax[row * n_tiles + tile] = mx;
    psum[row * n_tiles + tile] = ssum[0] + ssum[1] + ssum[2] + ssum[3];
    parg[row * n_tiles + tile] = arg;
  }
}

// the small tiles while the large ones would fill less than half of the 256 compute units (a 64 x 64 tile re-reads its
// operands a quarter as often, which counts once the chip is full)
static bool few_rows(const AcceptLaunch& a) {
  return (int64_t)((a.V + kTN - 1) / kTN) * ((a.plan.rows + kTM - 1) / kTM) < 128;
}

bool verify_front_supported(const AttnLaunch& at, const AcceptLaunch& a) {
  // where attention writes what the head reads (hidden states or W in attn_out), they run one after the other: the head sees the output
  const uintptr_t out = (uintptr_t)at.out, out_end = out + (size_t)at.B * at.Nq * at.Hq * at.D * sizeof(float);
  auto meets_out = [&](const void* p, size_t rows) {
    return (uintptr_t)p < out_end && out < (uintptr_t)p + rows * a.H * sizeof(float);
  };
  if (meets_out(a.hidden, (size_t)a.plan.rows) || meets_out(a.lm_head, (size_t)a.V)) return false;
  if (at.bf16 || at.kv_fp8 || at.lse_out || a.bf16 || a.fp8 || !few_rows(a)) return false;
  const int64_t wgs = (int64_t)at.B * at.Nq * at.Hq * at.plan.max_splits;
  // Long contexts, step in us as two launches and as one.  64-wide heads: the compiler keeps a K load less in flight in the shared
  // kernel, which past some four million (query row, token) pairs is more than the launch: 2 x 8 positions x 8 heads x 30 000 tokens 299.7,
  // 298.3; 7 x 8 x 8 x 17 000 527, 550; 9 x 10 x 8 x 30 000 1493, 1534 (128-wide: 11 x 6 x 16 x 13 000 2099, 1982).
  if (at.D == 64 && wgs * at.plan.split_len > (1 << 22)) return false;
  // Attention that would all be resident by itself, but is not behind the head's tiles, starts late: with splits of more than 512 tokens
  // (1 x 1 x 8 x 65 536 tokens of 128 and 8000 logits of 1024 204, 223; 1000 logits of 256, all resident, 185, 177), or where the
  // head's tiles alone take two rounds (128-wide heads: the shared kernel's registers leave room for three workgroups, the head's own for five) and
  // are long: 3 x 11 x 8 x 64 tokens and 8000 logits of 512, 1024, 2048, 4096: 45.4, 44.2; 57.8, 60.8; 85.7, 99.7; 143, 177.
  // More attention than that covers them: 8 x 8 x 8 x 900 and 6500 of 2048 159, 143.
  const int64_t resident = 256 * (at.D == 64 ? 5 : 3);
  const int64_t lm = (int64_t)((a.V + kSN - 1) / kSN) * ((a.plan.rows + kSM - 1) / kSM);
  if (wgs <= resident && wgs + lm > resident && (at.plan.split_len > 512 || (lm > resident && a.H > 1024))) return false;
  return wgs < (1 << 23);  // (one grid dimension holds the workgroups of both: fewer than 2^32 threads)
}

hipError_t launch_verify_front(const AttnLaunch& at, const AcceptLaunch& a, hipStream_t st) {
  const int lm_x = (a.V + kSN - 1) / kSN, lm_y = (int)((a.plan.rows + kSM - 1) / kSM);
  const bool whole = at.plan.max_splits == 1;
  const dim3 grid((unsigned)lm_x * lm_y + (unsigned)at.B * at.Nq * at.Hq * at.plan.max_splits);
  const size_t lds = (size_t)at.plan.split_len * (sizeof(float) + sizeof(uint32_t));
#define AURORA_FRONT(D, WHOLE)                                                                                               \
  hipLaunchKernelGGL((verify_front_f32<D, WHOLE>), grid, dim3(kGenThreads), lds, st, at, (const float*)a.hidden,              \
                     (const float*)a.lm_head, a.logits, a.plan.rows, a.H, a.V, lm_x, lm_y)
  if (at.D == 64) {
    if (whole) AURORA_FRONT(64, true); else AURORA_FRONT(64, false);
  } else {
    if (whole) AURORA_FRONT(128, true); else AURORA_FRONT(128, false);
  }
#undef AURORA_FRONT
  if (hipError_t e = hipGetLastError(); e != hipSuccess || whole) return e;
  return launch_attn_combine(at, st);
}

hipError_t launch_row_stats(const AcceptLaunch& a, hipStream_t st) {
  const float inv_t = a.temperature > 0.f ? 1.f / a.temperature : 1.f;
  hipLaunchKernelGGL(row_tile_stats, dim3(a.plan.n_tiles, (unsigned)a.plan.rows), dim3(256), 0, st, a.logits, a.pmax, a.psum,
                     a.parg, a.V, a.plan.stat_tile, a.plan.n_tiles, inv_t, a.temps, a.Nq);
  return hipGetLastError();
}

hipError_t launch_lmhead_generic(const AcceptLaunch& a, hipStream_t st) {
  const int64_t M = a.plan.rows;
  if (few_rows(a)) {
    dim3 grid((unsigned)((a.V + kSN - 1) / kSN), (unsigned)((M + kSM - 1) / kSM));
    if (a.bf16)
      hipLaunchKernelGGL(lmhead_generic_few<bf16_t>, grid, dim3(256), 0, st, (const bf16_t*)a.hidden,
                         (const bf16_t*)a.lm_head, a.logits, M, a.H, a.V);
    else
      hipLaunchKernelGGL(lmhead_generic_few<float>, grid, dim3(256), 0, st, (const float*)a.hidden,
                         (const float*)a.lm_head, a.logits, M, a.H, a.V);
  } else {
    dim3 grid((unsigned)((a.V + kTN - 1) / kTN), (unsigned)((M + kTM - 1) / kTM));
    if (a.bf16)
      hipLaunchKernelGGL(lmhead_generic<bf16_t>, grid, dim3(256), 0, st, (const bf16_t*)a.hidden,
                         (const bf16_t*)a.lm_head, a.logits, M, a.H, a.V);
    else
      hipLaunchKernelGGL(lmhead_generic<float>, grid, dim3(256), 0, st, (const float*)a.hidden,
                         (const float*)a.lm_head, a.logits, M, a.H, a.V);
  }
  return hipGetLastError();
}

}  // namespace aurora
