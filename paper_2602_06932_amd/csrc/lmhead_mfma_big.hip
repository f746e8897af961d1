// LM-head projection for many token rows (large batches, draft trees), where the contraction is bound by the matrix cores and
// by the way their operands take into LDS rather than by the sweep over W (appendix A.1, eq. 4 of the paper: target logits
// l in R^{T x V}; softmax statistics fused as in the small-M kernel).
//
// One workgroup of 8 wavefronts owns 256 vocabulary rows x 32 kT token rows (kT <= 8); wavefront (v, m) owns 64 vocab rows x
// 16 kT tokens (4 x kT accumulator tiles of 16 x 16).  The token rows of a call are cut into tiles of 32 and dealt evenly to
// the fewest workgroup columns, so a launch uses at most two values of kT, one apart (544 rows: 6 + 6 + 5).
//
// 16 x 16 products: v_mfma_f32_16x16x32_bf16 and v_mfma_scale_f32_16x16x128_f8f6f4.  On operands like these the part's power
// limit sets the rate, and under it the smaller form gets further than the 32x32x16 one: 1280 x 200064 x 6144 2820 -> 2680 us from
// the change of form alone.
//
// What bounds it then is latency: the vector cache returns a compute unit's loads in the order they were asked for, so a load
// that hits L2 waits behind W's misses in front of it, and how long a load may take is how long before its use it can leave,
// for all of them alike.  So loads leave in the order of their use, as soon as a piece of LDS falls free, in pieces half a
// stage long.  A stage is 128 bytes of each row (64 bf16 or 128 fp8 elements): W in a ring of three stages, the token rows in
// two rings of two, one for the first half of either token half's tiles and one for the rest.  A stage has two barriers, each
// one token tile after the products switch halves: the first opens half b (and frees half a and W, which have been read by
// then), the second opens W and half a of the next stage (and frees half b).  A token load has 1.5 stages to arrive, a W load
// 2 to 2.5.  With W asked for as early as three stages allowed, token rows one stage ahead and one barrier a stage, everything in
// flight had to drain at every barrier: 2680 us; now 2475 us (1.27 PFLOP/s; 512 x 128256 x 4096 520 -> 465 us, fp8 283 -> 262).
// Without any loads in its main loop the launch takes 2020 us, without the epilogue 2300; a 128 bytes wide prefetch of W's
// lines into L2 makes it slower (every prefetch is one more miss to wait behind), and so do rows of 64 bytes a stage.
//
// Operands roll through the registers: a stage's W fragments (32 registers) are read into a second set as the stage before
// ends, a token tile's fragment takes the registers of the one multiplied half a stage earlier.  The eight 16-byte chunks of a
// row segment are XOR-swizzled by (row / 2) mod 8 on the way in, which makes the 128-bit operand reads conflict free.
// kFp8: operands are E4M3 codes with one float32 scale per token row and per vocabulary row, applied to the accumulators in
// the epilogue.
#include "launch.hpp"
#include "lmhead_tile.hpp"

namespace aurora {

constexpr int kBgThreads = 512;
constexpr int kBgRowBytes = 128;                // bytes of a row segment per stage: 64 bf16 or 128 fp8 elements
constexpr int kBgVTile = 256;                   // vocab rows per workgroup (= statistics tile)
constexpr int kBgMTile = 256;                   // token rows per workgroup, at most
constexpr int kBgWBytes = kBgVTile * kBgRowBytes;      // 32 KB: a stage's W rows
constexpr int kBgHBytes = kBgMTile / 2 * kBgRowBytes;  // 16 KB: half of a stage's token rows
constexpr int kBgWStages = 3;
constexpr int kBgHStages = 2;
constexpr unsigned kBgNowhere = 0x40000000u;    // an offset past any descriptor: nothing is read, the LDS gets zeros
constexpr int kBgHRing = kBgWStages * kBgWBytes;       // token halves a of two stages, then halves b
constexpr int kBgLdsBytes = kBgHRing + 2 * kBgHStages * kBgHBytes;  // 160 KB

// Direct global->LDS load of 16 bytes per lane through a buffer descriptor; lane i's data lands at lds_base + 16 i.
// The address is descriptor base + voff (per lane, 32 bits) + soff (scalar); the hardware checks voff + soff against
// the descriptor's byte count (out-of-range lanes read zero and touch nothing).  Written as
// inline assembly so that the compiler does not order every later LDS read behind all such loads;
// the explicit vmcnt waits below do the waiting.  m0 holds the LDS base; one wait state is required
// between writing m0 and the load that reads it.
typedef __attribute__((ext_vector_type(4))) int i32x4_t;
template <bool kNonTemporal = false>
__device__ __forceinline__ void dma16(i32x4_t rsrc, unsigned voff, unsigned soff, unsigned lds_base) {
  if constexpr (kNonTemporal)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds" ::"s"(lds_base), "v"(voff),
                 "s"(rsrc), "s"(soff)
                 : "memory");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds_base), "v"(voff),
                 "s"(rsrc), "s"(soff)
                 : "memory");
}
// Raw buffer descriptor (stride 0) over `bytes` bytes at p; the words are made wave-uniform.
__device__ __forceinline__ i32x4_t bg_rsrc(const void* p, unsigned bytes) {
  const uint64_t a = (uint64_t)(uintptr_t)p;
  i32x4_t r;
  r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  r[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)((a >> 32) & 0xffffu));
  r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
  r[3] = 0x00020000;  // 32-bit data format, no swizzle, no index stride
  return r;
}

struct BgArgs {
  const char* hidden;
  const char* w;
  const float* h_scale;
  const float* w_scale;
  float* logits;
  float* pmax;
  float* psum;
  int32_t* parg;
  float* hmax;
  int M, H, V, n_tiles;
  float exp_scale;     // log2(e) / T
  const float* temps;  // per-request T, or NULL
  int Nq;
};

template <int P> struct BgParity { static constexpr int value = P; };

// One workgroup's tile: vocabulary tile vt, token rows m0 .. m0 + 32 kT.  kOne: one workgroup column holds all token rows.
template <bool kFp8, int kT, bool kOne>
__device__ __forceinline__ void bg_tile(const BgArgs& A, char* lds, int vt, int m0) {
  static_assert(kT >= 4, "a half of two tiles has room for the reads of W");
  constexpr int kTa = (kT + 1) / 2, kTb = kT / 2;  // token tiles of the halves a and b of a stage
  const char* __restrict__ hidden = A.hidden;
  const char* __restrict__ w = A.w;
  const float* __restrict__ h_scale = A.h_scale;
  const float* __restrict__ w_scale = A.w_scale;
  float* __restrict__ logits = A.logits;
  const int M = A.M, H = A.H, V = A.V, n_tiles = A.n_tiles, Nq = A.Nq;
  const float exp_scale = A.exp_scale;
  const float* __restrict__ temps = A.temps;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wvv = wave & 3;   // vocab slice of 64 rows
  const int wm = wave >> 2;   // token half
  const int vbase = vt * kBgVTile;
  const int mw = m0 + wm * 16 * kT;  // first token row of this wavefront
  constexpr int kEsz = kFp8 ? 1 : 2;  // bytes per operand element
  const int nk = H * kEsz / kBgRowBytes;
  const unsigned lds0 = (unsigned)(uintptr_t)lds;  // LDS pointers are 32-bit offsets

  // ---- loads: instruction i of an operand brings eight rows; a wavefront issues instructions wave and wave + 8 of each half
  // stage of W (128 rows) and of the token rows (the first kTa or the last kTb tiles of either token half), whatever exists of
  // them, so that the counts it waits for are constants.
  // The descriptors cover exactly the rows that exist: one past the end is zeros in LDS, and nothing is stored of it.
  const size_t row_bytes = (size_t)H * kEsz;
  const int v_here = V - vbase < kBgVTile ? V - vbase : kBgVTile, m_here = M - m0 < 32 * kT ? M - m0 : 32 * kT;
  const i32x4_t w_rsrc = bg_rsrc(w + (size_t)vbase * row_bytes, (unsigned)(v_here * row_bytes));
  const i32x4_t h_rsrc = bg_rsrc(hidden + (size_t)m0 * row_bytes, (unsigned)(m_here * row_bytes));
  const int lrow = lane >> 3, lslot = lane & 7;
  const int chunk = (lslot ^ ((8 * wave + lrow) >> 1 & 7)) * 16;  // (instruction i + 8 starts 64 rows further: same swizzle)
  unsigned w_off[4], h_off[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = 64 * j + 8 * wave + lrow;
    w_off[j] = (unsigned)(r * row_bytes + chunk);
    const int nh = 16 * (j < 2 ? kTa : kTb), ur = 64 * (j & 1) + 8 * wave + lrow;  // rows of a token half; row in the ring slot
    const int m = (j < 2 ? 0 : 16 * kTa) + (ur < nh ? ur : ur - nh + 16 * kT);
    h_off[j] = ur < 2 * nh ? (unsigned)(m * row_bytes + chunk) : kBgNowhere;
  }
  const unsigned lds_w = lds0 + 8 * wave * kBgRowBytes;
  // half `hf` of stage ks of W into ring slot offset `slot`; half hf of the token rows of stage ks
  // One column: its workgroups start their walk over the hidden dimension at different offsets and wrap around (rows are a
  // multiple of the memory-channel interleave apart: in lockstep all would ask the same channels; 128 rows 263 -> 205 us), and W, read
  // once, does not displace the token rows in L2.  Several columns walk in step: they share W's lines, and the columns of all
  // vocab tiles of an XCD their token rows (1280 rows staggered 2 % slower, 512 rows 1 %).  Below the rows where this kernel takes
  // every vocabulary, where either way is within 3 % of the other (bf16 in step ahead, fp8 staggered), the walk is staggered too:
  // the W-streaming kernel takes some vocabularies there, and a row's sums keep its order in both.
  const int k0 = kOne || M < kLmTiledOnlyRows ? (int)((vt * 13u) % (unsigned)nk) : 0;
  auto k_off = [&](int ks) { return ks < nk ? (unsigned)((ks + k0 >= nk ? ks + k0 - nk : ks + k0) * kBgRowBytes) : 0u; };
  auto issue_w = [&](int ks, unsigned slot, int hf) {
    const i32x4_t d = {w_rsrc[0], w_rsrc[1], ks < nk ? w_rsrc[2] : 0, w_rsrc[3]};  // past the end: nothing is read
#pragma unroll
    for (int j = 0; j < 2; ++j) dma16<kOne>(d, w_off[2 * hf + j], k_off(ks), lds_w + slot + 64 * (2 * hf + j) * kBgRowBytes);
  };
  auto issue_h = [&](int ks, int par, int hf) {
    const i32x4_t d = {h_rsrc[0], h_rsrc[1], ks < nk ? h_rsrc[2] : 0, h_rsrc[3]};
#pragma unroll
    for (int j = 0; j < 2; ++j)
      dma16(d, h_off[2 * hf + j], k_off(ks), lds_w + kBgHRing + (2 * hf + par) * kBgHBytes + 64 * j * kBgRowBytes);
  };

  const int li = lane & 31, lh = lane >> 5;
  // epilogue scratch, once the ring is done with: wavefront-private 8 KB each for turning the logits tiles, then [4][256]
  // statistics of the four vocab slices
  char* tb = lds + wave * 8192;
  float* st_max = (float*)(lds + 8 * 8192);
  float* st_sum = st_max + 4 * kBgMTile;
  int* st_arg = (int*)(st_sum + 4 * kBgMTile);
  float* st_half = (float*)(st_arg + 4 * kBgMTile);  // [8][256]: maxima of the eight groups of 32 vocab rows
  const int vrow0 = vbase + wvv * 64;
  const bool vec_ok = (V & 3) == 0;
  auto put_stats = [&](int col0, float mx, float sum, int arg, float half) {
    if (lh == 0) {
      st_max[wvv * kBgMTile + col0 + li] = mx;
      st_sum[wvv * kBgMTile + col0 + li] = sum;
      st_arg[wvv * kBgMTile + col0 + li] = arg;
    }
    st_half[(2 * wvv + lh) * kBgMTile + col0 + li] = half;
  };
  f32x4_t acc[kT][4];
#pragma unroll
  for (int u = 0; u < kT; ++u)
#pragma unroll
    for (int a = 0; a < 4; ++a) acc[u][a] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // An operand fragment is 32 bytes a lane: chunks lq and 4 + lq of row l15 - two bf16 steps of 32 elements, or one fp8 step of
  // 128 (which elements meet in which product does not matter as long as both operands are read the same way).
  typedef __attribute__((ext_vector_type(8))) int i32x8_t;
  const int l15 = lane & 15, lq = lane >> 4;
  const int c0 = (lq ^ (l15 >> 1)) * 16;  // the other chunk is 64 bytes across
  const char* wbase[2] = {lds + (wvv * 64 + l15) * kBgRowBytes + c0, lds + (wvv * 64 + l15) * kBgRowBytes + (c0 ^ 64)};
  const char* hbase[2] = {lds + kBgHRing + l15 * kBgRowBytes + c0,
                          lds + kBgHRing + l15 * kBgRowBytes + (c0 ^ 64)};
  auto read = [&](const char* const (&base)[2], int off, i32x8_t& f) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const i32x4_t v = *(const i32x4_t*)(base[e] + off);
#pragma unroll
      for (int i = 0; i < 4; ++i) f[4 * e + i] = v[i];
    }
  };
  i32x8_t wA[4], wB[4], hf[kTa];
  auto read_w = [&](unsigned slot, int a, i32x8_t& f) { read(wbase, (int)slot + a * 16 * kBgRowBytes, f); };
  // token tile u of a stage of parity par; a tile of half b takes the registers of the one of half a that has been multiplied
  auto read_h = [&](int par, int u) {
    const int b = u >= kTa, i = b ? u - kTa : u;
    read(hbase, (2 * b + par) * kBgHBytes + (wm * (b ? kTb : kTa) + i) * 16 * kBgRowBytes, hf[i]);
  };
  constexpr int kMul = kFp8 ? 4 : 8;  // products per token tile and stage
  auto multiply = [&](const i32x8_t (&wf)[4], int u) {
    const i32x8_t& h = hf[u < kTa ? u : u - kTa];
    if constexpr (kFp8) {
#pragma unroll
      for (int a = 0; a < 4; ++a)
        acc[u][a] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(wf[a], h, acc[u][a], 0, 0, 0, 127, 0, 127);
    } else {
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const i32x4_t wv = {wf[a][4 * e], wf[a][4 * e + 1], wf[a][4 * e + 2], wf[a][4 * e + 3]};
          const i32x4_t hv = {h[4 * e], h[4 * e + 1], h[4 * e + 2], h[4 * e + 3]};
          acc[u][a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wv), __builtin_bit_cast(bf16x8_t, hv),
                                                              acc[u][a], 0, 0, 0);
        }
    }
  };
  // every read of this wavefront is back before it says so to the others; its loads but the last `younger` have landed
#define BG_OPEN(younger)                                                    \
  do {                                                                      \
    __builtin_amdgcn_sched_barrier(0);                                      \
    __builtin_amdgcn_s_waitcnt((7 << 4) | (3 << 14) | 15); /* lgkmcnt(0) */ \
    LM_WAIT_VMCNT(younger);                                                 \
    __builtin_amdgcn_s_barrier();                                           \
    asm volatile("" ::: "memory");                                          \
    __builtin_amdgcn_sched_barrier(0);                                      \
  } while (0)
  unsigned s0 = 0, s1 = kBgWBytes, s2 = 2 * kBgWBytes;  // W ring slots of stages ks, ks + 1 and ks + 2
  auto stage = [&](int ks, auto parity, const i32x8_t (&wc)[4], i32x8_t (&wn)[4]) {
    constexpr int par = decltype(parity)::value;
#pragma unroll
    for (int u = 0; u < kT; ++u) {
      multiply(wc, u);
      int reads = 0;
      if (u == 0) {
        BG_OPEN(10);  // half b of stage ks is there; its half a and its W have been read
        issue_h(ks + 2, par, 0);
      }
      if (u == 1) issue_w(ks + 3, s0, 0);
      if (u == kTa) {
        BG_OPEN(10);  // W and half a of stage ks + 1 are there; half b of stage ks has been read
        issue_h(ks + 2, par, 1);
      }
      if (u == kTa + 1) issue_w(ks + 3, s0, 1);
      if (u < kTb) {
        read_h(par, u + kTa);
        reads += 2;
      }
      if (u >= kTa) {
        read_h(par ^ 1, u - kTa);
        reads += 2;
      }
      if (u == kTa && kTa > kTb) {
        read_h(par ^ 1, kTa - 1);
        reads += 2;
      }
#pragma unroll
      for (int a = 0; a < 4; ++a)
        if (u == kTa + a / 2) {
          read_w(s1, a, wn[a]);
          reads += 2;
        }
      if (u != 0 && u != kTa) __builtin_amdgcn_sched_group_barrier(0x008, kMul, 0);
      if (reads == 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      if (reads == 4) __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
      if (reads == 6) __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
      if (reads == 8) __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    const unsigned t = s0;
    s0 = s1;
    s1 = s2;
    s2 = t;
  };

  // what the stages before the first would have asked for, in their order
  issue_h(0, 0, 0);
  issue_w(0, 0, 0);
  issue_w(0, 0, 1);
  issue_w(1, kBgWBytes, 0);
  issue_h(0, 0, 1);
  issue_w(1, kBgWBytes, 1);
  issue_h(1, 1, 0);
  issue_w(2, 2 * kBgWBytes, 0);
  issue_h(1, 1, 1);
  issue_w(2, 2 * kBgWBytes, 1);
  BG_OPEN(14);
#pragma unroll
  for (int a = 0; a < 4; ++a) read_w(0, a, wA[a]);
#pragma unroll
  for (int u = 0; u < kTa; ++u) read_h(0, u);
  int ks = 0;
  for (; ks + 1 < nk; ks += 2) {
    stage(ks, BgParity<0>{}, wA, wB);
    stage(ks + 1, BgParity<1>{}, wB, wA);
  }
  if (ks < nk) stage(ks, BgParity<0>{}, wA, wB);
  LM_WAIT_VMCNT(0);  // (loads past the end write zeros)
  __syncthreads();   // every wavefront is done with the ring; it becomes epilogue scratch
#undef BG_OPEN

  if constexpr (kFp8) {
    // dequantise: accumulator (vocab row v, token m) times w_scale[v] * h_scale[m]
    float hs[kT];
#pragma unroll
    for (int u = 0; u < kT; ++u) {
      const int m = mw + 16 * u + l15;
      hs[u] = h_scale[m < M ? m : M - 1];
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int v = vrow0 + 16 * a + 4 * lq;  // four consecutive vocabulary rows
      float wsc[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) wsc[e] = w_scale[v + e < V ? v + e : V - 1];
#pragma unroll
      for (int u = 0; u < kT; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[u][a][e] *= wsc[e] * hs[u];
    }
  }
#pragma unroll
  for (int u = 0; u < kT; u += 2) {
    const int m = mw + 16 * u;
    if (m < M) {  // tiles wholly past the last token row hold nothing
      float mx, sum, half;
      int arg;
      const float es = lm_row_scale(exp_scale, temps, Nq, m + li, M);
      if (u + 1 < kT) lm_tile_out16<2>(&acc[u], vrow0, V, m, M, es, tb, logits, vec_ok, lane, mx, sum, arg, half);
      else lm_tile_out16<1>(&acc[u], vrow0, V, m, M, es, tb, logits, vec_ok, lane, mx, sum, arg, half);
      if (u + 1 < kT || li < 16) put_stats(m - m0, mx, sum, arg, half);
    }
  }
  __syncthreads();
  if (tid < 32 * kT) {
    const int m = m0 + tid;
    if (m < M) {
      float mx, sum;
      int arg;
      lm_merge_waves(st_max, st_sum, st_arg, kBgMTile, tid, lm_row_scale(exp_scale, temps, Nq, m, M), mx, sum, arg);
      const size_t o = (size_t)m * n_tiles + vt;
      A.pmax[o] = mx;
      A.psum[o] = sum;
      A.parg[o] = arg;
      // the eight group maxima of this tile, 32 contiguous bytes per token row
      f32x4_t h0, h1;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        h0[j] = st_half[j * kBgMTile + tid];
        h1[j] = st_half[(4 + j) * kBgMTile + tid];
      }
      f32x4_t* hd = (f32x4_t*)(A.hmax + o * kLmHalfPerTile);
      hd[0] = h0;
      hd[1] = h1;
    }
  }
}

// Workgroup columns [0, n_a) hold 32 kTA token rows each, the others 32 kTB (kTB = kTA or kTA - 1).
template <bool kFp8, int kTA, int kTB, bool kOne>
__global__ __launch_bounds__(kBgThreads, 1) void lmhead_mfma_big_kernel(BgArgs A, int m_tiles, int n_a) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  // Workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2.  The m_tiles token tiles
  // of one vocab tile get ids 8 apart: same XCD, launched together - the W tile comes from HBM once and
  // from L2 for the others.  Where they walk the hidden dimension in step (bg_tile), the
  // workgroups resident on one XCD want the same slices of the token tiles at about the same time
  // and its L2 serves all but the first.
  const int wg = blockIdx.x;
  const int vt = (wg / (8 * m_tiles)) * 8 + (wg & 7);
  const int mt = (wg >> 3) % m_tiles;
  if (vt >= A.n_tiles) return;
  if constexpr (kTA == kTB) {
    bg_tile<kFp8, kTA, kOne>(A, lds, vt, mt * 32 * kTA);
  } else {
    if (mt < n_a) bg_tile<kFp8, kTA, kOne>(A, lds, vt, mt * 32 * kTA);
    else bg_tile<kFp8, kTB, kOne>(A, lds, vt, n_a * 32 * kTA + (mt - n_a) * 32 * kTB);
  }
}

bool lmhead_mfma_big_supported(const AcceptLaunch& a) {
  const int esz = a.fp8 ? 1 : 2;
  return (a.bf16 || a.fp8) && (a.H * esz) % kBgRowBytes == 0 && a.H * esz >= kBgRowBytes &&
         a.H * esz <= (1 << 20) /* 256 rows of a tile within a 32-bit buffer offset */ && a.V >= 1 &&
         a.plan.stat_tile == kBgVTile;
}

template <bool kFp8, int kTA, int kTB, bool kOne>
static hipError_t launch_big_t(const AcceptLaunch& a, hipStream_t st, int m_tiles, int n_a) {
  static LdsAttrOnce attr;
  if (hipError_t e = attr.ensure((const void*)lmhead_mfma_big_kernel<kFp8, kTA, kTB, kOne>, kBgLdsBytes); e != hipSuccess)
    return e;
  BgArgs A = {};
  A.hidden = (const char*)a.hidden; A.w = (const char*)a.lm_head; A.h_scale = a.hidden_scale; A.w_scale = a.lm_scale;
  A.logits = a.logits; A.pmax = a.pmax; A.psum = a.psum; A.parg = a.parg; A.hmax = a.hmax;
  A.M = (int)a.plan.rows; A.H = a.H; A.V = a.V; A.n_tiles = a.plan.n_tiles;
  A.exp_scale = 1.4426950408889634f / (a.temperature > 0.f ? a.temperature : 1.f);
  A.temps = a.temps; A.Nq = a.Nq;
  const int v_tiles = (a.V + kBgVTile - 1) / kBgVTile;
  dim3 grid((v_tiles + 7) / 8 * 8 * m_tiles);
  hipLaunchKernelGGL((lmhead_mfma_big_kernel<kFp8, kTA, kTB, kOne>), grid, dim3(kBgThreads), kBgLdsBytes, st, A, m_tiles, n_a);
  return hipGetLastError();
}

// Tiles of 32 token rows dealt evenly to the fewest workgroup columns of at most eight.
void lmhead_mfma_big_geometry(int M, int* m_tiles, int* nt_a, int* nt_b, int* n_a) {
  const int tiles = (M + 31) / 32;
  const int cols = (tiles + 7) / 8;
  const int base = tiles / cols, rem = tiles % cols;
  *m_tiles = cols;
  *nt_a = rem ? base + 1 : base;
  *nt_b = base;
  *n_a = rem ? rem : cols;
}

template <bool kFp8>
static hipError_t launch_big_dt(const AcceptLaunch& a, hipStream_t st) {
  int m_tiles, nta, ntb, n_a;
  lmhead_mfma_big_geometry((int)a.plan.rows, &m_tiles, &nta, &ntb, &n_a);
  // (what tiled_is_ahead lets through: one column of 129 to 256 rows, or eleven tiles and more in several)
  switch (m_tiles == 1 ? nta : nta * 10 + ntb) {
    case 5: return launch_big_t<kFp8, 5, 5, true>(a, st, m_tiles, n_a);
    case 6: return launch_big_t<kFp8, 6, 6, true>(a, st, m_tiles, n_a);
    case 7: return launch_big_t<kFp8, 7, 7, true>(a, st, m_tiles, n_a);
    case 8: return launch_big_t<kFp8, 8, 8, true>(a, st, m_tiles, n_a);
    case 65: return launch_big_t<kFp8, 6, 5, false>(a, st, m_tiles, n_a);
    case 66: return launch_big_t<kFp8, 6, 6, false>(a, st, m_tiles, n_a);
    case 76: return launch_big_t<kFp8, 7, 6, false>(a, st, m_tiles, n_a);
    case 77: return launch_big_t<kFp8, 7, 7, false>(a, st, m_tiles, n_a);
    case 87: return launch_big_t<kFp8, 8, 7, false>(a, st, m_tiles, n_a);
    case 88: return launch_big_t<kFp8, 8, 8, false>(a, st, m_tiles, n_a);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_lmhead_mfma_big(const AcceptLaunch& a, hipStream_t st) {
  return a.fp8 ? launch_big_dt<true>(a, st) : launch_big_dt<false>(a, st);
}

}  // namespace aurora
