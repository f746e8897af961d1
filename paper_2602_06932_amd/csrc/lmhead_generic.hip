// Generic LM-head projection (fp32 FMA, fp32 or bf16 storage) followed by per-tile softmax
// statistics.  It is the fp32 path of the library and the fallback for shapes the MFMA kernel
// does not cover.  logits[m, v] = sum_h hidden[m, h] * W[v, h]  (appendix A.1, eq. 4: l in R^{T x V}).
#include "common.hpp"
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

// The same product for few token rows: 64 x 64 tiles would leave most of the chip idle (16 workgroups on 20 x 1024) and walk
// the hidden dimension in steps of 16 with two barriers each.  Here a workgroup takes 16 vocabulary rows x 32 token rows and
// 64 hidden elements per step, the next step's operands being loaded into registers (16 bytes a thread) while the present
// ones are multiplied out of LDS; a thread owns one vocabulary row and two token rows.  20 x 1024 x 256 in fp32: 25 -> 6 us.
constexpr int kSM = 32, kSN = 16, kSK = 64, kSPad = 4;
template <typename T>
__global__ __launch_bounds__(256) void lmhead_generic_few(const T* __restrict__ hidden, const T* __restrict__ w,
                                                          float* __restrict__ logits, int64_t M, int H, int V) {
  typedef __attribute__((ext_vector_type(4))) float f32x4_t;
  __shared__ __attribute__((aligned(16))) float As[kSM][kSK + kSPad];
  __shared__ __attribute__((aligned(16))) float Bs[kSN][kSK + kSPad];
  const int tid = threadIdx.x;
  const int v0 = blockIdx.x * kSN;
  const int64_t m0 = (int64_t)blockIdx.y * kSM;
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

hipError_t launch_lmhead_generic(const AcceptLaunch& a, hipStream_t st) {
  const int64_t M = a.plan.rows;
  // the small tiles while the large ones would fill less than half of the 256 compute units (a 64 x 64 tile re-reads its
  // operands a quarter as often, which counts once the chip is full)
  const int64_t large = (int64_t)((a.V + kTN - 1) / kTN) * ((M + kTM - 1) / kTM);
  if (large < 128) {
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
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const float inv_t = a.temperature > 0.f ? 1.f / a.temperature : 1.f;
  hipLaunchKernelGGL(row_tile_stats, dim3(a.plan.n_tiles, (unsigned)M), dim3(256), 0, st, a.logits, a.pmax, a.psum,
                     a.parg, a.V, a.plan.stat_tile, a.plan.n_tiles, inv_t, a.temps, a.Nq);
  return hipGetLastError();
}

}  // namespace aurora
