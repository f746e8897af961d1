// bf16 chunk attention on the matrix cores (paper sections 3.1 / 3.2: the Nq draft positions of a
// request - a chain, or a tree under its ancestor mask - are verified in one pass over the cached
// context).  head_dim 128, KV pages of 16 * 2^i tokens.
//
// The KV sweep is cut into 32-token tiles of one (request, KV head) pair; the tiles of the whole batch,
// numbered request-major, are dealt out in equal contiguous runs to a fixed number of resident
// workgroups (two per compute unit), whatever the mix of sequence lengths - over few tokens (build_split in
// attn_tile.hpp) a workgroup takes a few tiles of one pair.  A workgroup's run meets one or a few pairs; for each it produces one partial (m, l, O) - a "segment" - that a small merge
// kernel folds.  The G*Nq query rows that share a KV head form the 32-wide N side of
// v_mfma_f32_32x32x16_bf16, so a KV byte is read once for the whole GQA group.  Inside a segment the
// four wavefronts are independent: wavefront w owns every 4th tile, with private LDS buffers, a
// private online-softmax state, and no workgroup barrier until the segment's merge.
//
//   S^T = K Q^T   tokens are MFMA rows, query rows MFMA columns: a lane owns ONE query row and
//                 16 tokens, so max / sum reduce inside the lane plus one cross-half exchange, and
//                 the exp'd scores are already laid out as the B operand of the next product;
//   O^T = V^T P^T again one query row per lane, so the running rescale is lane-local.
//
// K and V tiles (32 tokens x 256 B) come in by direct global->LDS loads, 16 B per lane, each
// instruction covering four whole token rows (fully coalesced); chunks are XOR-swizzled by
// (row mod 8) so that both the 128-bit K operand reads and the 16-bit strided V^T reads are
// bank-conflict free.  K(t+1) is requested as soon as S(t) has consumed K(t), V(t+1) after
// O += P V(t), so HBM requests stay in flight through the softmax and MFMA phases.
#include "launch.hpp"
#include "attn_tile.hpp"

#include <algorithm>

namespace aurora {

// Units of work are 32-token tiles of one (request, KV head) pair, numbered request-major.  PB[b] is
// the number of units before request b; PB[B] the total.
__global__ __launch_bounds__(256) void attn_plan_kernel(const int32_t* __restrict__ seq_lens, int B, int Hkv,
                                                        int32_t* __restrict__ PB) {
  __shared__ int s_part[256];
  __shared__ int s_carry;
  const int tid = threadIdx.x;
  if (tid == 0) { s_carry = 0; PB[0] = 0; }
  __syncthreads();
  for (int b0 = 0; b0 < B; b0 += 256) {
    const int b = b0 + tid;
    const int mine = b < B ? ((seq_lens[b] + kAtTile - 1) / kAtTile) * Hkv : 0;
    s_part[tid] = mine;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {  // inclusive scan
      const int v = tid >= o ? s_part[tid - o] : 0;
      __syncthreads();
      s_part[tid] += v;
      __syncthreads();
    }
    if (b < B) PB[b + 1] = s_carry + s_part[tid];
    __syncthreads();
    if (tid == 255) s_carry += s_part[255];
    __syncthreads();
  }
}

hipError_t launch_attn_plan(const int32_t* seq_lens, int B, int Hkv, int32_t* PB, hipStream_t st) {
  hipLaunchKernelGGL(attn_plan_kernel, dim3(1), dim3(256), 0, st, seq_lens, B, Hkv, PB);
  return hipGetLastError();
}

constexpr int kNarrowPar = 4;  // tiles of a run that the narrow kernel's wavefronts take at a time
constexpr int kWidePar = 2;    // ... the wide kernel's two tile-parity groups

// kFp8KV: kp_ / vp_ hold E4M3 codes and k_scale / v_scale [Hkv] their per-head scales; they too go straight into LDS and are
// widened between the LDS read and the matrix instruction (see attn_tile.hpp).  Staged through registers and widened into
// LDS the sweep of 32 requests of 1K-4K tokens took 53 us (the loads in flight, the accumulators and the conversions did not
// fit into 256 registers: every tile waited for spill traffic behind its loads); with codes in LDS 37 us, 4.2 TB/s.
template <bool kLocalPlan, bool kFp8KV>
__global__ __launch_bounds__(kAtThreads, 2) void attn_mfma_kernel(
    const bf16_t* __restrict__ q, const void* __restrict__ kp_, const void* __restrict__ vp_,
    const float* __restrict__ k_scale, const float* __restrict__ v_scale,
    const int32_t* __restrict__ block_table, const int32_t* __restrict__ seq_lens,
    const int32_t* __restrict__ parents, int32_t* __restrict__ PB, float* __restrict__ part_o,
    float* __restrict__ part_ml, int B, int Nq, int Hq, int Hkv, int page_shift, int max_pages, float scale_log2_q) {
  const bf16_t* kp = (const bf16_t*)kp_;
  const bf16_t* vp = (const bf16_t*)vp_;
  // K and V tiles live in separate LDS objects: the compiler tracks pending LDS-direct loads per object,
  // so a read of a K tile does not wait for the V tile still in flight (and vice versa)
  __shared__ __attribute__((aligned(1024))) char kbuf_all[4 * kAtTileBytes];
  __shared__ __attribute__((aligned(1024))) char vbuf_all[4 * kAtTileBytes];
  __shared__ __attribute__((aligned(1024))) char qbuf[32 * kAtRowBytes];  // the segment's 32 query rows
  __shared__ float s_m[4][32];
  __shared__ float s_l[4][32];

  __shared__ int s_pb[kLocalPlan ? kLocalPlanMax + 1 : 1];
  __shared__ int2 s_wsum[4];
  __shared__ int s_par[kMaxNq];  // the request's tree: the ancestor walk is a chain of dependent reads
  __shared__ int4 s_first;
  SplitLens lens;
  if constexpr (kLocalPlan) lens = load_split_lens(seq_lens, B);
  auto pbv = [&](int i) -> int { return kLocalPlan ? s_pb[i] : PB[i]; };
  const int rt = blockIdx.y, row_tiles = gridDim.y;

  const int G = Hq / Hkv;
  const int R = G * Nq;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 31, lh = lane >> 5;
  char* kbuf = kbuf_all + wv * kAtTileBytes;
  char* vbuf = vbuf_all + wv * kAtTileBytes;

  // this lane's query row (MFMA column li) within the group: node n, head g
  const int mrow = rt * 32 + li;
  const bool row_ok = mrow < R;
  const int node = row_ok ? mrow / G : 0;
  // the query row this thread stages into LDS at the start of a segment (8 threads per row, 32 B each)
  const int qs_row = tid >> 3;
  const int qs_m = rt * 32 + qs_row;
  const bool qs_ok = qs_m < R;
  const int qs_node = qs_ok ? qs_m / G : 0;
  const int qs_g = qs_ok ? qs_m % G : 0;

  Share sh;
  if constexpr (kLocalPlan) {
    // every workgroup builds the split itself; the first one also publishes it for the merge kernel
    sh = build_split<kAtThreads, kNarrowPar, kAttnWorkgroups>(lens, B, Hkv, s_pb, s_wsum, &s_first);
    if (blockIdx.x == 0 && blockIdx.y == 0) publish_split(PB, s_pb, B, sh.by_run, kAtThreads);
  } else {
    sh = load_split<kAttnWorkgroups>(PB, seq_lens, B);
  }
  const bool by_run = sh.by_run;
  int u = sh.u, b = sh.b, from = sh.from, to = sh.to, L_next = sh.L;
  const int u_end = sh.u_end;
  if (u >= u_end) return;

  // ---- one segment per (request, KV head) pair this workgroup's unit range touches --------------------
  while (u < u_end) {
    while (to <= u) {
      from = to;
      to = pbv(++b + 1);
    }
    const int L = L_next;
    const int n_b = (L + kAtTile - 1) / kAtTile;
    const int rel = u - from;
    const int per_pair = by_run ? (n_b + kNarrowPar - 1) / kNarrowPar : n_b;
    const int hk = __builtin_amdgcn_readfirstlane(rel / per_pair);
    const int at = rel - hk * per_pair;
    const int t0 = by_run ? at * kNarrowPar : at;
    const int t1 = min(n_b, t0 + (by_run ? kNarrowPar : u_end - u));
    const int slot = blockIdx.x + b * Hkv + hk;  // segments are a monotone path in (workgroup, pair): unique
    u += by_run ? 1 : t1 - t0;
    if (u < u_end) {  // the next segment's length, under this one
      int bn = b;
      while (pbv(bn + 1) <= u) ++bn;
      L_next = seq_lens[bn];
    }

    const int start = t0 * kAtTile;
    const int prefix = L - Nq;
    const float scale_log2 = kFp8KV ? scale_log2_q * k_scale[hk] : scale_log2_q;
    // the segment's 32 query rows: on their way while the first tiles are requested
    const u32x4_t* qp = (const u32x4_t*)(q + (((size_t)b * Nq + qs_node) * Hq + hk * G + qs_g) * kAtD);
    const int c0 = (tid & 7) * 2;
    const u32x4_t qz = {0u, 0u, 0u, 0u};
    const u32x4_t q0 = qs_ok ? qp[c0] : qz;
    const u32x4_t q1 = qs_ok ? qp[c0 + 1] : qz;
    const int par_n = parents && tid < Nq ? parents[(size_t)b * Nq + tid] : -1;
    const int ntile = t1 - t0;
    const int32_t* bt = block_table + (size_t)b * max_pages;

    // Tile loads: always exactly 8 instructions of 4 token rows each (the s_waitcnt bookkeeping below
    // counts them).  Rows past the end of the sequence re-read the last valid token; their scores are
    // masked to -inf, so their (finite) values are multiplied by exact zeros.  A 32-token tile touches
    // at most two pages, whose ids are fetched with scalar loads.
    auto tile_pages = [&](int tt, int& pid_a, int& pid_b) {
      const int j0 = start + tt * kAtTile;
      pid_a = bt[j0 >> page_shift];
      pid_b = bt[min(j0 + 16, L - 1) >> page_shift];
    };
    auto issue_k = [&](int tt, int pid_a, int pid_b) {
      const int j0 = start + tt * kAtTile;
#pragma unroll
      for (int j = 0; j < 8; ++j) issue_rows<false>(kp, kbuf, j, j0, L, page_shift, Hkv, hk, pid_a, pid_b, lane);
    };
    auto issue_v = [&](int tt, int pid_a, int pid_b) {
      const int j0 = start + tt * kAtTile;
#pragma unroll
      for (int j = 0; j < 8; ++j) issue_rows<true>(vp, vbuf, j, j0, L, page_shift, Hkv, hk, pid_a, pid_b, lane);
    };

    SoftmaxState st;
    softmax_state_reset(st);

    // query rows -> LDS, 16-byte chunks swizzled like the K rows (they are read the same way)
    auto stage_query = [&]() {
      *(u32x4_t*)(qbuf + qs_row * kAtRowBytes + ((c0 ^ (qs_row & 15)) * 16)) = q0;
      *(u32x4_t*)(qbuf + qs_row * kAtRowBytes + (((c0 + 1) ^ (qs_row & 15)) * 16)) = q1;
      if (tid < Nq) s_par[tid] = par_n;
      __syncthreads();
    };
    if constexpr (kFp8KV) {
      // This wavefront's tiles are wv, wv + 4, ...; K and V of two of them are on their way into the two halves of its
      // buffers, and tile i + 2 takes the place of tile i as soon as the products have read it.
      const int n_my = ntile > wv ? (ntile - wv + 3) >> 2 : 0;
      const uint8_t* kp8 = (const uint8_t*)kp_;
      const uint8_t* vp8 = (const uint8_t*)vp_;
      auto issue_k8 = [&](int i, int pid_a, int pid_b) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          issue_rows8<false>(kp8, kbuf + (i & 1) * kAtTile8, j, start + (wv + 4 * i) * kAtTile, L, page_shift, Hkv, hk, pid_a,
                             pid_b, lane);
      };
      auto issue_v8 = [&](int i, int pid_a, int pid_b) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          issue_rows8<true>(vp8, vbuf + (i & 1) * kAtTile8, j, start + (wv + 4 * i) * kAtTile, L, page_shift, Hkv, hk, pid_a,
                            pid_b, lane);
      };
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (i < n_my) {
          int pa, pb;
          tile_pages(wv + 4 * i, pa, pb);
          issue_k8(i, pa, pb);
          issue_v8(i, pa, pb);
        }
      stage_query();
      const unsigned long long anc = ancestor_mask(parents ? s_par : nullptr, node, Nq);
      QFrags qf;
      load_q_frags8(qf, qbuf, li, lh);
      for (int i = 0; i < n_my; ++i) {
        const bool next = i + 1 < n_my, more = i + 2 < n_my;
        int pa = 0, pb = 0;  // page ids of tile i + 2: scalar loads issued a tile ahead of their use
        if (more) tile_pages(wv + 4 * (i + 2), pa, pb);
        if (next) WAIT_VMCNT(12); else WAIT_VMCNT(4);  // K(i) landed; V(i), K(i+1), V(i+1) may be in flight
        const f32x16_t s_acc = tile_scores8(kbuf + (i & 1) * kAtTile8, qf, li, lh);
        asm volatile("" ::: "memory");  // the LDS reads above stay above the overwrite
        if (more) issue_k8(i + 2, pa, pb);
        bf16x8_t pb2[2];
        tile_softmax(s_acc, st, pb2, scale_log2, start + (wv + 4 * i) * kAtTile, prefix, L, anc, lh);
        if (more) WAIT_VMCNT(12); else if (next) WAIT_VMCNT(8); else WAIT_VMCNT(0);  // V(i) landed
        tile_pv8(vbuf + (i & 1) * kAtTile8, pb2, st, lane);
        asm volatile("" ::: "memory");
        if (more) issue_v8(i + 2, pa, pb);
      }
    } else {
    int tt = wv;
    if (tt < ntile) {
      int pa0, pb0;
      tile_pages(tt, pa0, pb0);
      issue_k(tt, pa0, pb0);
      issue_v(tt, pa0, pb0);
    }
    stage_query();
    // chunk slots this node may see: itself and its ancestors (chain: every slot up to its own)
    const unsigned long long anc = ancestor_mask(parents ? s_par : nullptr, node, Nq);
    for (; tt < ntile; tt += 4) {
      const bool more = tt + 4 < ntile;
      // page ids of the next tile: scalar loads issued a whole tile ahead of their use
      int npa = 0, npb = 0;
      if (more) tile_pages(tt + 4, npa, npb);
      WAIT_VMCNT(8);  // K(t) landed (V(t) may still be in flight)
      const f32x16_t s_acc = tile_scores(kbuf, qbuf, li, lh);
      // the K buffer is free once the products above have their operands; the memory clobber keeps
      // the compiler from moving the LDS reads below the overwrite
      asm volatile("" ::: "memory");
      if (more) issue_k(tt + 4, npa, npb);
      bf16x8_t pb2[2];
      tile_softmax(s_acc, st, pb2, scale_log2, start + tt * kAtTile, prefix, L, anc, lh);
      if (more) WAIT_VMCNT(8); else WAIT_VMCNT(0);  // V(t) landed (K(t+1) may be in flight)
      tile_pv(vbuf, pb2, st, lane);
      asm volatile("" ::: "memory");
      if (more) issue_v(tt + 4, npa, npb);
    }
    }
    f32x16_t(&o_acc)[4] = st.o;
    const float m_run = st.m_run, l_half = st.l_half;

    // ---- merge the four wavefronts and write this segment's partial (m, l, O) -------------------------
    float l_row = l_half + __shfl_xor(l_half, 32, kWave);
    if (lh == 0) { s_m[wv][li] = m_run; s_l[wv][li] = l_row; }
    __syncthreads();  // also: every wavefront is done with its K/V buffers
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) M = fmaxf(M, s_m[w][li]);
    const float M_safe = M == -INFINITY ? 0.f : M;
    float l_tot = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) l_tot += s_l[w][li] * __builtin_amdgcn_exp2f(s_m[w][li] - M_safe);
    const float f_own = __builtin_amdgcn_exp2f(m_run - M_safe) * (kFp8KV ? v_scale[hk] : 1.f);
    // each wavefront parks its rescaled O^T as [row li][64 d] floats in its K buffer (columns 0..63)
    // and its V buffer (columns 64..127)
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      float* obuf = (float*)((db < 2 ? kbuf_all : vbuf_all) + wv * kAtTileBytes);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int dd = 32 * (db & 1) + 8 * g + 4 * lh;  // column within the 64-wide half
        f32x4_t o = {o_acc[db][4 * g] * f_own, o_acc[db][4 * g + 1] * f_own, o_acc[db][4 * g + 2] * f_own,
                     o_acc[db][4 * g + 3] * f_own};
        if (m_run == -INFINITY) o = f32x4_t{0.f, 0.f, 0.f, 0.f};  // nothing visible: 0 x infinity must not get in
        // rotate the 16-byte slot by the row so that the 32 rows of a column group spread over banks
        *(f32x4_t*)(obuf + li * 64 + ((dd / 4 + li) & 15) * 4) = o;
      }
    }
    __syncthreads();
    // wavefront w sums and stores d-block w (32 columns) of all rows
    {
      const int db = wv;
      const size_t prow = ((size_t)slot * row_tiles + rt) * 32 + li;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int dd = 32 * (db & 1) + 8 * g + 4 * lh;
        f32x4_t sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const float* ob = (const float*)((db < 2 ? kbuf_all : vbuf_all) + w * kAtTileBytes);
          sum += *(const f32x4_t*)(ob + li * 64 + ((dd / 4 + li) & 15) * 4);
        }
        if (row_ok) *(f32x4_t*)(part_o + prow * kAtD + 32 * db + 8 * g + 4 * lh) = sum;
      }
      if (row_ok && wv == 0 && lh == 0) {
        part_ml[prow * 2 + 0] = M * (1.0f / kLog2e);  // natural-log units
        part_ml[prow * 2 + 1] = l_tot;
      }
    }
    __syncthreads();  // the K/V buffers are about to be refilled for the next segment
  }
}

// ---- wide-row variant: more than 32 query rows per (request, KV head) pair (draft trees) ----------------
// Eight wavefronts: wavefront (g, w) owns the 32-row query tile w and the KV tiles of parity g, so a KV
// byte is still read once per pair while two wavefronts per SIMD hide each other's latencies.  K/V
// tiles go through a ring of LDS stages of two tiles each (every wavefront loads an eighth of both),
// one workgroup barrier per step; one workgroup per compute unit.  Work is dealt out exactly as in the
// narrow kernel; a segment ends with a merge of the two parities through LDS.
constexpr int kWideThreads = 512;
constexpr int kWideWorkgroups = 256;  // one per compute unit
constexpr int kWideStages = 3;
constexpr int kWideStageBytes = 2 * 2 * kAtTileBytes;                // two tiles, K and V
constexpr int kWideQBytes = 4 * 32 * kAtRowBytes;                    // four query tiles
constexpr int kWideLdsBytes = kWideQBytes + kWideStages * kWideStageBytes;

// kFp8KV: the cache holds E4M3 codes, which go into the ring as they are and are widened behind the LDS read, as in the
// narrow kernel: a stage is half as large, so the ring holds twice as many.  16 trees of 32 nodes over 4096 tokens: sweep 69 us
// with codes staged in registers and widened into the ring -> 59 us; 20 trees of 45 nodes, 0.9K-7K: 174 -> 153 us.
constexpr int kWide8Stages = 6;
constexpr int kWide8StageBytes = 2 * 2 * kAtTile8;
static_assert(kWide8Stages == 6 && kWide8Stages * kWide8StageBytes <= kWideStages * kWideStageBytes, "the ring's bytes");
template <bool kLocalPlan, bool kFp8KV>
__global__ __launch_bounds__(kWideThreads, 1) void attn_mfma_wide_kernel(
    const bf16_t* __restrict__ q, const void* __restrict__ kp_, const void* __restrict__ vp_,
    const float* __restrict__ k_scale, const float* __restrict__ v_scale,
    const int32_t* __restrict__ block_table, const int32_t* __restrict__ seq_lens,
    const int32_t* __restrict__ parents, int32_t* __restrict__ PB, float* __restrict__ part_o,
    float* __restrict__ part_ml, int B, int Nq, int Hq, int Hkv, int page_shift, int max_pages, int row_tiles,
    float scale_log2_q) {
  const bf16_t* kp = (const bf16_t*)kp_;
  const bf16_t* vp = (const bf16_t*)vp_;
  extern __shared__ __attribute__((aligned(1024))) char wlds[];
  char* qall = wlds;
  char* ring = wlds + kWideQBytes;
  __shared__ int s_pb[kLocalPlan ? kLocalPlanMax + 1 : 1];
  __shared__ int2 s_wsum[kWideThreads / kWave];
  __shared__ int s_par[kMaxNq];
  __shared__ float s_ml[2][4][2][32];  // (m, l) of the rows of each parity group's query tiles
  __shared__ int4 s_first;
  SplitLens lens;
  if constexpr (kLocalPlan) lens = load_split_lens(seq_lens, B);
  auto pbv = [&](int i) -> int { return kLocalPlan ? s_pb[i] : PB[i]; };

  const int G = Hq / Hkv;
  const int R = G * Nq;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2, wq = wave & 3;
  const int li = lane & 31, lh = lane >> 5;
  const int rt = blockIdx.y * 4 + wq;          // this wavefront's query tile
  const bool rt_ok = rt < row_tiles;           // wave-uniform
  const int mrow = rt * 32 + li;
  const bool row_ok = rt_ok && mrow < R;
  const int node = row_ok ? mrow / G : 0;
  const char* qtile = qall + wq * (32 * kAtRowBytes);
  const int qs_row = (tid & 255) >> 3;  // staging: 8 threads per query row, 32 B each
  const int qs_half = tid >> 8;         // threads 0..255 stage tiles 0 and 1, threads 256..511 tiles 2 and 3

  Share sh;
  if constexpr (kLocalPlan) {
    // every workgroup builds the split itself; the first one also publishes it for the merge kernel
    sh = build_split<kWideThreads, kWidePar, kWideWorkgroups>(lens, B, Hkv, s_pb, s_wsum, &s_first);
    if (blockIdx.x == 0 && blockIdx.y == 0) publish_split(PB, s_pb, B, sh.by_run, kWideThreads);
  } else {
    sh = load_split<kWideWorkgroups>(PB, seq_lens, B);
  }
  const bool by_run = sh.by_run;
  int u = sh.u, b = sh.b, from = sh.from, to = sh.to, L_next = sh.L;
  const int u_end = sh.u_end;
  if (u >= u_end) return;

  while (u < u_end) {
    while (to <= u) {
      from = to;
      to = pbv(++b + 1);
    }
    const int L = L_next;
    const int n_b = (L + kAtTile - 1) / kAtTile;
    const int rel = u - from;
    const int per_pair = by_run ? (n_b + kWidePar - 1) / kWidePar : n_b;
    const int hk = __builtin_amdgcn_readfirstlane(rel / per_pair);
    const int at = rel - hk * per_pair;
    const int t0 = by_run ? at * kWidePar : at;
    const int t1 = min(n_b, t0 + (by_run ? kWidePar : u_end - u));
    const int slot = blockIdx.x + b * Hkv + hk;
    u += by_run ? 1 : t1 - t0;
    if (u < u_end) {  // the next segment's length, under this one
      int bn = b;
      while (pbv(bn + 1) <= u) ++bn;
      L_next = seq_lens[bn];
    }
    const int start = t0 * kAtTile;
    const int prefix = L - Nq;
    const int ntile = t1 - t0;
    const int nstep = (ntile + 1) >> 1;
    const int last_tile_start = ((L - 1) >> 5) << 5;
    const int32_t* bt = block_table + (size_t)b * max_pages;
    const float scale_log2 = kFp8KV ? scale_log2_q * k_scale[hk] : scale_log2_q;

    // the four query tiles: on their way while the first steps are requested
    const int c0 = (tid & 7) * 2;
    u32x4_t q0[2], q1[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int m = (blockIdx.y * 4 + qs_half * 2 + i) * 32 + qs_row;
      const bool ok = m < R;
      const int nd = ok ? m / G : 0, g = ok ? m % G : 0;
      const u32x4_t* qp = (const u32x4_t*)(q + (((size_t)b * Nq + nd) * Hq + hk * G + g) * kAtD);
      const u32x4_t z = {0u, 0u, 0u, 0u};
      q0[i] = ok ? qp[c0] : z;
      q1[i] = ok ? qp[c0 + 1] : z;
    }
    const int par_n = parents && tid < Nq ? parents[(size_t)b * Nq + tid] : -1;

    // this wavefront's eighth of a step: load instruction `wave` of K and of V, for both tiles of the step
    // (a tile past the end of the sequence re-reads the last one; it is never multiplied)
    // page ids of the step's two tiles: scalar loads, a step ahead of their use
    int pid[2][2];
    auto j0_of = [&](int sidx, int g) { return min(start + (2 * sidx + g) * kAtTile, last_tile_start); };
    auto fetch_pages = [&](int sidx) {
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        pid[g][0] = bt[j0_of(sidx, g) >> page_shift];
        pid[g][1] = bt[min(j0_of(sidx, g) + 16, L - 1) >> page_shift];
      }
    };
    auto issue_step = [&](int sidx) {
      char* stage = ring + (sidx % kWideStages) * kWideStageBytes;
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        char* kb = stage + g * (2 * kAtTileBytes);
        issue_rows<false>(kp, kb, wave, j0_of(sidx, g), L, page_shift, Hkv, hk, pid[g][0], pid[g][1], lane);
        issue_rows<true>(vp, kb + kAtTileBytes, wave, j0_of(sidx, g), L, page_shift, Hkv, hk, pid[g][0], pid[g][1], lane);
      }
    };

    SoftmaxState st;
    softmax_state_reset(st);
    QFrags qf;  // this wavefront's query tile as MFMA operand fragments, for the whole run
    unsigned long long anc;
    auto stage_query = [&]() {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        char* dst = qall + (qs_half * 2 + i) * (32 * kAtRowBytes) + qs_row * kAtRowBytes;
        *(u32x4_t*)(dst + ((c0 ^ (qs_row & 15)) * 16)) = q0[i];
        *(u32x4_t*)(dst + (((c0 + 1) ^ (qs_row & 15)) * 16)) = q1[i];
      }
      if (tid < Nq) s_par[tid] = par_n;
      __syncthreads();
      if constexpr (kFp8KV) load_q_frags8(qf, qtile, li, lh); else load_q_frags(qf, qtile, li, lh);
      anc = ancestor_mask(parents ? s_par : nullptr, node, Nq);
    };
    if constexpr (kFp8KV) {
      // a wavefront's eighth of a step: eight token rows of K and of V of one of the step's two tiles
      const uint8_t* kp8 = (const uint8_t*)kp_;
      const uint8_t* vp8 = (const uint8_t*)vp_;
      auto issue_step8 = [&](int sidx) {
        char* kb = ring + (sidx % kWide8Stages) * kWide8StageBytes + grp * (2 * kAtTile8);
        const int j0 = min(start + (2 * sidx + grp) * kAtTile, last_tile_start);
        const int pid_a = bt[j0 >> page_shift];
        const int pid_b = bt[min(j0 + 16, L - 1) >> page_shift];
        issue_rows8<false>(kp8, kb, wq, j0, L, page_shift, Hkv, hk, pid_a, pid_b, lane);
        issue_rows8<true>(vp8, kb + kAtTile8, wq, j0, L, page_shift, Hkv, hk, pid_a, pid_b, lane);
      };
      for (int i = 0; i < kWide8Stages - 1 && i < nstep; ++i) issue_step8(i);
      stage_query();
      for (int sidx = 0; sidx < nstep; ++sidx) {
        // steps sidx+1 .. sidx+kWide8Stages-2 may stay in flight; near the end of the segment fewer were issued
        const int younger = nstep - 1 - sidx;
        if (younger >= 4) WAIT_VMCNT(8);
        else if (younger == 3) WAIT_VMCNT(6);
        else if (younger == 2) WAIT_VMCNT(4);
        else if (younger == 1) WAIT_VMCNT(2);
        else WAIT_VMCNT(0);
        __builtin_amdgcn_s_barrier();  // step complete from all eight wavefronts; the previous step's stage is free
        asm volatile("" ::: "memory");
        if (sidx + kWide8Stages - 1 < nstep) issue_step8(sidx + kWide8Stages - 1);
        const int tt = 2 * sidx + grp;
        if (rt_ok && tt < ntile) {
          const char* kb = ring + (sidx % kWide8Stages) * kWide8StageBytes + grp * (2 * kAtTile8);
          const f32x16_t s_acc = tile_scores8(kb, qf, li, lh);
          bf16x8_t pb2[2];
          tile_softmax(s_acc, st, pb2, scale_log2, start + tt * kAtTile, prefix, L, anc, lh);
          tile_pv8(kb + kAtTile8, pb2, st, lane);
        }
        asm volatile("" ::: "memory");
      }
    } else {
      for (int i = 0; i < kWideStages - 1 && i < nstep; ++i) {
        fetch_pages(i);
        issue_step(i);
      }
      fetch_pages(kWideStages - 1);
      stage_query();
      for (int sidx = 0; sidx < nstep; ++sidx) {
        // steps sidx+1 .. sidx+kWideStages-2 may stay in flight; near the end of the segment fewer were issued
        if (nstep - 1 - sidx >= kWideStages - 2) WAIT_VMCNT(4 * (kWideStages - 2)); else WAIT_VMCNT(0);
        __builtin_amdgcn_s_barrier();  // step complete from all eight wavefronts; the previous step's stage is free
        asm volatile("" ::: "memory");
        if (sidx + kWideStages - 1 < nstep) {  // (after the scores' products instead: 2 to 4 % slower)
          issue_step(sidx + kWideStages - 1);
          fetch_pages(sidx + kWideStages);
        }
        const int tt = 2 * sidx + grp;
        if (rt_ok && tt < ntile) {
          const char* kb = ring + (sidx % kWideStages) * kWideStageBytes + grp * (2 * kAtTileBytes);
          const f32x16_t s_acc = tile_scores_qreg(kb, qf, li, lh);
          bf16x8_t pb2[2];
          tile_softmax(s_acc, st, pb2, scale_log2, start + tt * kAtTile, prefix, L, anc, lh);
          tile_pv(kb + kAtTileBytes, pb2, st, lane);
        }
        asm volatile("" ::: "memory");
      }
    }

    pin_accumulators(st);
    // The two parity groups' results of a query tile become one partial: each group hands half of its columns to the
    // other through the idle ring (lane-linear, the lanes of both hold the same rows), so that a segment writes 512
    // bytes per query row and the merge kernel reads as many.
    const float l_row = st.l_half + __shfl_xor(st.l_half, 32, kWave);
    __syncthreads();  // every wavefront is done with the ring
    if (lh == 0) { s_ml[grp][wq][0][li] = st.m_run; s_ml[grp][wq][1][li] = l_row; }
    f32x4_t* give = (f32x4_t*)(ring + wave * kAtTileBytes) + lane;
    const f32x4_t* take = (const f32x4_t*)(ring + (wave ^ 4) * kAtTileBytes) + lane;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x16_t& src = grp == 0 ? st.o[2 + db] : st.o[db];
        give[(db * 4 + g) * kWave] = f32x4_t{src[4 * g], src[4 * g + 1], src[4 * g + 2], src[4 * g + 3]};
      }
    __syncthreads();
    const float m_own = st.m_run, m_oth = s_ml[grp ^ 1][wq][0][li], l_oth = s_ml[grp ^ 1][wq][1][li];
    const float m_new = fmaxf(m_own, m_oth), m_ref = m_new == -INFINITY ? 0.f : m_new;
    const float f_own = __builtin_amdgcn_exp2f(m_own - m_ref), f_oth = __builtin_amdgcn_exp2f(m_oth - m_ref);
    if (row_ok) {
      const size_t prow = ((size_t)slot * row_tiles + rt) * 32 + li;
      const float vs = kFp8KV ? v_scale[hk] : 1.f;
#pragma unroll
      for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x16_t& src = grp == 0 ? st.o[db] : st.o[2 + db];
          // (a group in whose tiles the row saw nothing counts for nothing, also where its sums are 0 x infinity)
          const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
          f32x4_t own = {src[4 * g], src[4 * g + 1], src[4 * g + 2], src[4 * g + 3]};
          f32x4_t oth = take[(db * 4 + g) * kWave];
          if (m_own == -INFINITY) own = z;
          if (m_oth == -INFINITY) oth = z;
          const f32x4_t o = own * (f_own * vs) + oth * (f_oth * vs);
          *(f32x4_t*)(part_o + prow * kAtD + 32 * (2 * grp + db) + 8 * g + 4 * lh) = o;
        }
      if (grp == 0 && lh == 0) {
        part_ml[prow * 2 + 0] = m_new * (1.0f / kLog2e);  // natural-log units (-inf if nothing was visible)
        part_ml[prow * 2 + 1] = f_own * l_row + f_oth * l_oth;
      }
    }
    __syncthreads();  // the query tiles and the ring are about to be rewritten
  }
}

// Merge the partials of one output row (request b, node n, query head hq): the segments of its
// (request, KV head) pair sit in slots w + pair for the workgroups w whose unit range meets the pair's.
// Thirty-two threads (four output columns each) fold a run of a row's partials, a few at a time: the merge is a short
// chain of dependent loads, so what counts is how many loads are in flight.  A row is given to kSplit such groups of
// threads, whose results meet in LDS; a workgroup is eight groups.  One request of 2777 tokens: 27 us with 64
// partials a row, one row per group and four partials at a time -> 4.1 us with 22 partials, one per run, and kSplit = 8.
constexpr int kCombineGroups = 8;
template <int kSplit>
__global__ __launch_bounds__(32 * kCombineGroups) void attn_mfma_combine(const float* __restrict__ part_o,
                                                                         const float* __restrict__ part_ml,
                                                                         const int32_t* __restrict__ seq_lens,
                                                                         const int32_t* __restrict__ PB,
                                                                         bf16_t* __restrict__ out, int B, int Nq, int Hq,
                                                                         int Hkv, int wgs, int row_tiles,
                                                                         int par, float* __restrict__ lse_out) {
  const int grp = threadIdx.x >> 5, sub = grp % kSplit;
  const int b = blockIdx.x / Nq, n = blockIdx.x - b * Nq;
  const int hq = blockIdx.y * (kCombineGroups / kSplit) + grp / kSplit;
  const size_t row = (size_t)blockIdx.x * Hq + hq;  // (b*Nq + n)*Hq + hq
  const bool row_ok = hq < Hq;
  if (kSplit == 1 && !row_ok) return;
  const int d4 = threadIdx.x & 31;  // columns 4 d4 .. 4 d4 + 3
  float M = -INFINITY, den = 0.f;
  f32x4_t num = {0.f, 0.f, 0.f, 0.f};
  if (row_ok) {
    const int G = Hq / Hkv;
    const int hk = hq / G;
    const int mrow = n * G + hq - hk * G;
    const int rt = mrow >> 5, li = mrow & 31;
    const int n_b = (seq_lens[b] + kAtTile - 1) / kAtTile;
    int w0, np;
    pair_owners(PB, B, b, hk, n_b, wgs, par, w0, np);
    const int pair = b * Hkv + hk;
    const int per = (np + kSplit - 1) / kSplit;
    const int p_end = min(np, (sub + 1) * per);
    const size_t prow0 = ((size_t)(w0 + pair) * row_tiles + rt) * 32 + li;
    constexpr int kU = kSplit == 1 ? 4 : 8;
    for (int p0 = sub * per; p0 < p_end; p0 += kU) {
      float ms[kU], ls[kU];
      f32x4_t os[kU];
      float top = -INFINITY;
#pragma unroll
      for (int i = 0; i < kU; ++i) {
        const bool ok = p0 + i < p_end;
        const size_t prow = prow0 + (size_t)(ok ? p0 + i : p0) * row_tiles * 32;
        const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
        ms[i] = ok ? part_ml[prow * 2] : -INFINITY;
        ls[i] = ok ? part_ml[prow * 2 + 1] : 0.f;
        os[i] = ok ? *(const f32x4_t*)(part_o + prow * kAtD + 4 * d4) : z;
        top = fmaxf(top, ms[i]);
      }
      const float nm = fmaxf(M, top);
      if (nm == -INFINITY) continue;  // nothing visible so far
      const float fo = __expf(M - nm);
      num *= fo;
      den *= fo;
#pragma unroll
      for (int i = 0; i < kU; ++i) {
        // a partial with nothing visible is left out: its factor is exp(-inf) = 0, but its sums may be 0 x infinity
        const float fn = __expf(ms[i] - nm);
        if (ms[i] > -INFINITY) num += os[i] * fn;
        den += ls[i] * fn;
      }
      M = nm;
    }
  }
  if constexpr (kSplit > 1) {
    __shared__ float s_m[kCombineGroups], s_den[kCombineGroups];
    __shared__ f32x4_t s_num[kCombineGroups][32];
    s_num[grp][d4] = num;
    if (d4 == 0) { s_m[grp] = M; s_den[grp] = den; }
    __syncthreads();
    if (sub != 0 || !row_ok) return;
#pragma unroll
    for (int i = 1; i < kSplit; ++i) M = fmaxf(M, s_m[grp + i]);
    if (M > -INFINITY) {
      const float f0 = __expf(s_m[grp] - M);
      num *= f0;
      den *= f0;
#pragma unroll
      for (int i = 1; i < kSplit; ++i) {
        const float f = __expf(s_m[grp + i] - M);
        num += s_num[grp + i][d4] * f;
        den += s_den[grp + i] * f;
      }
    }
  }
  if (lse_out && d4 == 0) lse_out[row] = den > 0.f ? M + __logf(den) : -INFINITY;
  typedef __attribute__((ext_vector_type(4))) unsigned short u16x4_t;
  u16x4_t o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = f32_to_bf16(den > 0.f ? num[e] / den : 0.f);
  *(u16x4_t*)(out + row * kAtD + 4 * d4) = o;
}

template <int kSplit>
static void launch_combine(const AttnLaunch& a, hipStream_t st, int wgs, int row_tiles) {
  constexpr unsigned per_wg = kCombineGroups / kSplit;
  hipLaunchKernelGGL(attn_mfma_combine<kSplit>, dim3(a.B * a.Nq, (a.Hq + per_wg - 1) / per_wg), dim3(32 * kCombineGroups), 0,
                     st, a.part_o, a.part_ml, a.seq_lens, a.plan_pb, (bf16_t*)a.out, a.B, a.Nq, a.Hq, a.Hkv, wgs, row_tiles,
                     row_tiles == 1 ? kNarrowPar : kWidePar, a.lse_out);
}

bool attn_mfma_supported(const AttnLaunch& a) {
  return a.bf16 && a.D == kAtD && a.page >= 16 && (a.page & (a.page - 1)) == 0;
}

hipError_t launch_attn_mfma(const AttnLaunch& a, hipStream_t st) {
  const int R = a.Hq / a.Hkv * a.Nq;
  const int row_tiles = (R + 31) / 32;
  const bool local_plan = a.B <= kLocalPlanMax;
  hipError_t e;
  if (!local_plan) {
    e = launch_attn_plan(a.seq_lens, a.B, a.Hkv, a.plan_pb, st);
    if (e != hipSuccess) return e;
  }
  const int shift = __builtin_ctz(a.page);
  const float sc = a.scale * kLog2e;
  int wgs;
  if (row_tiles == 1) {
    wgs = kAttnWorkgroups;
    dim3 grid(wgs, 1);
#define AURORA_LAUNCH_NARROW(LOCAL, FP8)                                                                            \
  hipLaunchKernelGGL((attn_mfma_kernel<LOCAL, FP8>), grid, dim3(kAtThreads), 0, st, (const bf16_t*)a.q, a.k, a.v,    \
                     a.k_scale, a.v_scale, a.block_table, a.seq_lens, a.parents, a.plan_pb, a.part_o, a.part_ml, a.B, \
                     a.Nq, a.Hq, a.Hkv, shift, a.max_pages, sc)
    if (local_plan) {
      if (a.kv_fp8) AURORA_LAUNCH_NARROW(true, true); else AURORA_LAUNCH_NARROW(true, false);
    } else {
      if (a.kv_fp8) AURORA_LAUNCH_NARROW(false, true); else AURORA_LAUNCH_NARROW(false, false);
    }
#undef AURORA_LAUNCH_NARROW
  } else {
    wgs = kWideWorkgroups;
    dim3 grid(wgs, (row_tiles + 3) / 4);
#define AURORA_LAUNCH_WIDE(LOCAL, FP8)                                                                             \
  do {                                                                                                              \
    static LdsAttrOnce attr;                                                                                        \
    e = attr.ensure((const void*)attn_mfma_wide_kernel<LOCAL, FP8>, kWideLdsBytes);                                 \
    if (e != hipSuccess) return e;                                                                                  \
    hipLaunchKernelGGL((attn_mfma_wide_kernel<LOCAL, FP8>), grid, dim3(kWideThreads), kWideLdsBytes, st,            \
                       (const bf16_t*)a.q, a.k, a.v, a.k_scale, a.v_scale, a.block_table, a.seq_lens, a.parents,    \
                       a.plan_pb, a.part_o, a.part_ml, a.B, a.Nq, a.Hq, a.Hkv, shift, a.max_pages, row_tiles, sc);  \
  } while (0)
    if (local_plan) {
      if (a.kv_fp8) AURORA_LAUNCH_WIDE(true, true); else AURORA_LAUNCH_WIDE(true, false);
    } else {
      if (a.kv_fp8) AURORA_LAUNCH_WIDE(false, true); else AURORA_LAUNCH_WIDE(false, false);
    }
#undef AURORA_LAUNCH_WIDE
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  // Partials of a row if the requests are about equally long, and at most one per run of the longest that fits the block table.
  // From a dozen on, splitting a row over all groups of a workgroup shortens the chain (4.1 against 13 us at 22 partials);
  // below it the eight times as many workgroups cost more than the one or two rounds of loads they save (4096 rows of nine
  // partials: 13.0 split, 6.9 whole).
  const int64_t most = ((int64_t)a.max_pages * a.page + kAtTile - 1) / kAtTile / (row_tiles == 1 ? kNarrowPar : kWidePar) + 2;
  const int per_row = (int)std::min<int64_t>(wgs / (a.B * a.Hkv) + 1, most);
  if (per_row >= 12) launch_combine<8>(a, st, wgs, row_tiles);
  else launch_combine<1>(a, st, wgs, row_tiles);
  return hipGetLastError();
}

}  // namespace aurora
