// Pieces shared by the matrix-core attention kernels (forward and backward): operand types, the direct
// global->LDS tile loads, the work split into 32-token tiles, and the per-tile products.
#pragma once
#include "common.hpp"

namespace aurora {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(8))) unsigned short u16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_t;

constexpr int kAtThreads = 256;
constexpr int kAtD = 128;
constexpr int kAtTile = 32;                       // tokens per tile
constexpr int kAtRowBytes = kAtD * 2;             // 256
constexpr int kAtTileBytes = kAtTile * kAtRowBytes;  // 8 KB
constexpr float kLog2e = 1.4426950408889634f;

// Direct global->LDS load of 16 bytes per lane: lane i's data lands at lds_base + 16*i.  Written as
// inline assembly so that the compiler's own wait-count bookkeeping does not see it (it would make
// every later LDS read wait for ALL such loads); the explicit s_waitcnt vmcnt(n) below do the
// waiting.  Waits the compiler inserts for its own vector memory operations can only become more
// conservative, because the counter retires in order.
__device__ __forceinline__ void load_to_lds_16(const void* gptr, const void* lds_base) {
  const unsigned base = (unsigned)(uintptr_t)lds_base;  // LDS pointers are 32-bit offsets
  // m0 holds the LDS base; one wait state is required between writing m0 and the load that reads it.
  // Nothing else in this kernel uses m0.
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" ::"s"(__builtin_amdgcn_readfirstlane(base)),
               "v"(gptr)
               : "memory");
}
#define WAIT_VMCNT(n)                                                                              \
  do {                                                                                             \
    __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | (7 << 4) | (15 << 8));            \
    asm volatile("" ::: "memory");                                                                 \
  } while (0)

// The sweeps deal the U units to the workgroups as evenly as they divide: contiguous runs of U / wgs units, one
// more for the first U % wgs workgroups - every workgroup has work (if there is enough) and no compute unit holds more than its share.
__device__ __forceinline__ int unit_begin(int U, int wgs, int w) {
  const int q = U / wgs, r = U % wgs;
  return w * q + (w < r ? w : r);
}
// the workgroup whose run holds unit u (0 <= u < U)
__device__ __forceinline__ int unit_owner(int U, int wgs, int u) {
  const int q = U / wgs, r = U % wgs;
  const int edge = r * (q + 1);  // units below it sit in runs of q + 1
  return u < edge ? u / (q + 1) : r + (u - edge) / q;  // u >= edge implies q >= 1
}

// ---- pieces shared by the two sweep kernels -----------------------------------------------------------
struct SoftmaxState {
  f32x16_t o[4];   // O^T accumulators: block db, register r <-> column 32 db + 8(r/4) + 4*lh + r%4
  float m_run;     // running max of the scaled scores of this lane's query row, log2 units
  float l_half;    // running sum over the tokens this half-lane owns
};

__device__ __forceinline__ void softmax_state_reset(SoftmaxState& st) {
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) st.o[db][r] = 0.f;
  st.m_run = -INFINITY;
  st.l_half = 0.f;
}

// Chunk slots node n may see: itself and its ancestors (par: the request's parents, in LDS; NULL is a chain, where that is
// every slot up to its own).
__device__ __forceinline__ unsigned long long ancestor_mask(const int* par, int n, int Nq) {
  if (!par) return n == 63 ? ~0ull : ((1ull << (n + 1)) - 1);
  unsigned long long anc = 0;
  for (int a = n, hops = 0; a >= 0 && hops <= Nq; a = par[a], ++hops) anc |= 1ull << a;
  return anc;
}

// Placed between a tile loop and the code that consumes the accumulators piecewise: the accumulators leave the
// loop as four whole 16-register values.  Without it the compiler keeps a second, scattered copy of all 64
// registers for the later piecewise reads and refreshes it after the MFMAs of EVERY tile (64 moves per tile,
// and 36 more registers).
__device__ __forceinline__ void pin_accumulators(SoftmaxState& st) {
  asm volatile("" : "+v"(st.o[0]), "+v"(st.o[1]), "+v"(st.o[2]), "+v"(st.o[3]));
}

// Scores (register r <-> token j0 + 8(r/4) + 4 lh + r%4) of tokens that the lane's row does not see become -inf: past the prefix
// it sees the chunk slots of anc.  The tile's 32 tokens are formed as one word of bits (the tile reaches past the prefix, and the
// sequence past the tile's start); a test per token took sixteen branches, each with a saved execution mask.
__device__ __forceinline__ void mask_scores(f32x16_t& s_acc, int j0, int prefix, int L, unsigned long long anc, int lh) {
  const int before = prefix - j0, left = L - j0;  // tokens of the prefix, of the sequence
  unsigned seen = before > 0 ? ((unsigned)anc << before) | ((1u << before) - 1u) : (unsigned)(anc >> -before);
  if (left < kAtTile) seen &= (1u << left) - 1u;
  seen >>= 4 * lh;
#pragma unroll
  for (int r = 0; r < 16; ++r) s_acc[r] = seen & (1u << (8 * (r >> 2) + (r & 3))) ? s_acc[r] : -INFINITY;
}

// S^T = K Q^T for one 32-token tile: tokens are MFMA rows, the 32 query rows MFMA columns
__device__ __forceinline__ f32x16_t tile_scores(const char* kbuf, const char* qtile, int li, int lh) {
  f32x16_t s_acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) s_acc[r] = 0.f;
  const int sw = li & 15;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int coff = li * kAtRowBytes + (((2 * s + lh) ^ sw) * 16);
    const bf16x8_t ka = *(const bf16x8_t*)(kbuf + coff);
    const bf16x8_t qa = *(const bf16x8_t*)(qtile + coff);
    s_acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qa, s_acc, 0, 0, 0);
  }
  return s_acc;
}

// The same product with the query tile's operand fragments already in registers (32 VGPRs, loaded once per run of
// tiles by load_q_frags): a third less LDS traffic per tile.
struct QFrags { bf16x8_t f[8]; };
__device__ __forceinline__ void load_q_frags(QFrags& qf, const char* qtile, int li, int lh) {
  const int sw = li & 15;
#pragma unroll
  for (int s = 0; s < 8; ++s) qf.f[s] = *(const bf16x8_t*)(qtile + li * kAtRowBytes + (((2 * s + lh) ^ sw) * 16));
}
__device__ __forceinline__ f32x16_t tile_scores_qreg(const char* kbuf, const QFrags& qf, int li, int lh) {
  f32x16_t s_acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) s_acc[r] = 0.f;
  const int sw = li & 15;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const bf16x8_t ka = *(const bf16x8_t*)(kbuf + li * kAtRowBytes + (((2 * s + lh) ^ sw) * 16));
    s_acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qf.f[s], s_acc, 0, 0, 0);
  }
  return s_acc;
}

typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(4))) short s16x4_t;

// The running reference of a row's scaled scores only moves when a tile's maximum exceeds it by more
// than 2^kLazyBits: exp'd scores stay below 2^kLazyBits (exact in fp32, same relative rounding in
// bf16), and on most tiles no accumulator needs rescaling.
constexpr float kLazyBits = 8.0f;

// LDS position of 16-byte chunk c of V-tile row r: chunk ^ v_key(r).  Four consecutive token rows land in
// four different 64-byte groups, which is what the transposing reads below need to be conflict-free.
__device__ __forceinline__ int v_key(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }

// online softmax of the tile (register r holds token j0 + 8(r/4) + 4*lh + r%4 of this lane's row);
// returns the exp'd scores rounded to bf16 (hardware round-to-nearest-even), already laid out as the
// B operand of the P.V product.  The mask without branches and the halves meeting by a register exchange instead of a trip
// through LDS: 20 trees of 45 nodes over 0.9K to 7K tokens 167 -> 162 us, 16 of 32 over 4096 72 -> 67, on an 8-bit cache 62.4 -> 59.3;
// one request 12.1 -> 11.9.
__device__ __forceinline__ void tile_softmax(f32x16_t s_acc, SoftmaxState& st, bf16x8_t pb2[2], float scale_log2, int j0,
                                             int prefix, int L, unsigned long long anc, int lh) {
  if (j0 + kAtTile > prefix) mask_scores(s_acc, j0, prefix, L, anc, lh);
  float tmax = -INFINITY;
#pragma unroll
  for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, s_acc[r]);
  const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(tmax), __float_as_uint(tmax), false, false);
  tmax = fmaxf(__uint_as_float(halves[0]), __uint_as_float(halves[1])) * scale_log2;  // scale > 0: the max commutes with it
  if (__any(tmax > st.m_run + kLazyBits)) {  // wave-uniform branch
    const float m_new = tmax > st.m_run + kLazyBits ? tmax : st.m_run;
    const float alpha = __builtin_amdgcn_exp2f(st.m_run - (m_new == -INFINITY ? 0.f : m_new));
    st.m_run = m_new;
    st.l_half *= alpha;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) st.o[db][r] *= alpha;
  }
  const float neg_m = st.m_run == -INFINITY ? 0.f : -st.m_run;
  float psum = 0.f;
#pragma unroll
  for (int r = 0; r < 16; r += 2) {
    const float p0 = __builtin_amdgcn_exp2f(fmaf(s_acc[r], scale_log2, neg_m));
    const float p1 = __builtin_amdgcn_exp2f(fmaf(s_acc[r + 1], scale_log2, neg_m));
    psum += p0 + p1;
    const f32x2_t pp = {p0, p1};
    const bf16x2_t pk = __builtin_convertvector(pp, bf16x2_t);
    pb2[r >> 3][r & 7] = pk[0];
    pb2[r >> 3][(r & 7) + 1] = pk[1];
  }
  st.l_half += psum;
}

// O^T += V^T P^T.  The A operand needs, per lane, one column of V for eight tokens: two transposing LDS
// reads (ds_read_b64_tr_b16: within 16 lanes, lane i receives element i%4 of the 8-byte vectors
// addressed by lanes i/4, 4+i/4, 8+i/4, 12+i/4) fetch four tokens each.  Lane k of a 16-lane group
// therefore addresses token row tb + k/4, columns 4(k%4)..4(k%4)+3 of the group's 16 columns.
__device__ __forceinline__ void tile_pv(const char* vbuf, const bf16x8_t pb2[2], SoftmaxState& st, int lane) {
  const int lh = lane >> 5, k = lane & 15, kq = k >> 2;
  const int g1 = (lane >> 4) & 1;  // which 16 of the 32 columns of a block
  // byte address = row*256 + ((chunk ^ v_key(row)) * 16) + (col % 8) * 2 with
  //   row = 16u + 8e + 4lh + kq,  col = 32db + 16g1 + 4(k%4)   (see v_key; derivation in comments below)
  // v_key(row) = (kq << 2) | ((2e + lh) & 3);  chunk = 4db + 2g1 + (k%4)/2
  const int lo0 = ((2 * g1 + ((k & 3) >> 1)) ^ (lh & 3)) * 16;
  const int lo1 = ((2 * g1 + ((k & 3) >> 1)) ^ ((2 + lh) & 3)) * 16;
  const int common = lh * 1024 + kq * 256 + (k & 1) * 8 + kq * 64;
  const int base0 = common + lo0;          // e = 0
  const int base1 = common + lo1 + 2048;   // e = 1 (token rows + 8)
#pragma unroll
  for (int uu = 0; uu < 2; ++uu) {
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      typedef __attribute__((address_space(3))) s16x4_t* lds_v4;
      const s16x4_t r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(vbuf + uu * 4096 + (base0 ^ (db * 64))));
      const s16x4_t r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(vbuf + uu * 4096 + (base1 ^ (db * 64))));
      const u16x8_t va = {(unsigned short)r0[0], (unsigned short)r0[1], (unsigned short)r0[2], (unsigned short)r0[3],
                          (unsigned short)r1[0], (unsigned short)r1[1], (unsigned short)r1[2], (unsigned short)r1[3]};
      st.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, va), pb2[uu], st.o[db], 0, 0, 0);
    }
  }
}

// one of the 8 load instructions of a K or V tile: token rows 4j .. 4j+3 of the tile starting at j0
template <bool kIsV>
__device__ __forceinline__ void issue_rows(const bf16_t* pool, char* buf, int j, int j0, int L, int page_shift, int Hkv,
                                           int hk, int pid_a, int pid_b, int lane) {
  const int lrow = lane >> 4, lpos = lane & 15;
  const int pa = j0 >> page_shift;
  const int tok = min(j0 + 4 * j + lrow, L - 1);
  const int pid = (tok >> page_shift) == pa ? pid_a : pid_b;
  const int r = 4 * j + lrow;
  const int chunk = lpos ^ (kIsV ? v_key(r) : (r & 15));
  const bf16_t* src =
      pool + ((((size_t)pid * Hkv + hk) << page_shift) + (tok & ((1 << page_shift) - 1))) * kAtD + chunk * 8;
  load_to_lds_16(src, buf + j * 1024);
}

// ---- KV cache held as E4M3 codes (one byte per element, one scale per KV head) ----------------------------
// A 32-token tile of codes is 32 rows x 128 B = 4 KB each of K and V.  Both kernels bring the codes into LDS as
// they are and widens them to bf16 (exactly) between the LDS read and the matrix instruction: half the LDS bytes of a
// bf16 tile and no registers for tiles on their way.  The scales are applied outside the products: K's folds into the
// softmax scale, V's multiplies the segment's partial O.
constexpr int kAtRow8 = kAtD;                  // bytes of a token row of codes
constexpr int kAtTile8 = kAtTile * kAtRow8;    // 4 KB

// LDS position of 16-byte chunk c of row r: c ^ key.  K rows are read sixteen at a time, one chunk each (key (r >> 1) & 7
// puts them into different bank groups); a transposing V read takes 32 bytes of rows {0-3, 8-11} or {4-7, 12-15}, and rows
// of equal parity share a 128-byte bank half, whose four 32-byte slots the key deals out.
__device__ __forceinline__ int k8_key(int r) { return (r >> 1) & 7; }
__device__ __forceinline__ int v8_key(int r) { return (((r >> 1) & 1) | (((r >> 3) & 1) << 1)) << 1; }

// one of the 4 load instructions of a K or V tile of codes: token rows 8j .. 8j+7 of the tile starting at j0
template <bool kIsV>
__device__ __forceinline__ void issue_rows8(const uint8_t* pool, char* buf, int j, int j0, int L, int page_shift, int Hkv,
                                            int hk, int pid_a, int pid_b, int lane) {
  const int r = 8 * j + (lane >> 3);
  const int tok = min(j0 + r, L - 1);
  const int pid = (tok >> page_shift) == (j0 >> page_shift) ? pid_a : pid_b;
  const int chunk = (lane & 7) ^ (kIsV ? v8_key(r) : k8_key(r));
  const uint8_t* src =
      pool + ((((size_t)pid * Hkv + hk) << page_shift) + (tok & ((1 << page_shift) - 1))) * kAtRow8 + chunk * 16;
  load_to_lds_16(src, buf + j * 1024);
}

// eight E4M3 codes -> eight bf16 (exact: 3 mantissa bits and the exponent range fit)
__device__ __forceinline__ bf16x8_t widen8(unsigned lo, unsigned hi) {
  const u32x4_t w = {__builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, false)),
                     __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, true)),
                     __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, false)),
                     __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, true))};
  return __builtin_bit_cast(bf16x8_t, w);
}

// S^T = K Q^T from a tile of codes: lane half lh takes the sixteen codes 32 j + 16 lh .. of its token row for the products
// 2j and 2j + 1, so the query fragments are read in the same order.
__device__ __forceinline__ void load_q_frags8(QFrags& qf, const char* qtile, int li, int lh) {
#pragma unroll
  for (int s = 0; s < 8; ++s)
    qf.f[s] = *(const bf16x8_t*)(qtile + li * kAtRowBytes + (((4 * (s >> 1) + 2 * lh + (s & 1)) ^ (li & 15)) * 16));
}
__device__ __forceinline__ f32x16_t tile_scores8(const char* kbuf, const QFrags& qf, int li, int lh) {
  f32x16_t s_acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) s_acc[r] = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const u32x4_t c = *(const u32x4_t*)(kbuf + li * kAtRow8 + (((2 * j + lh) ^ k8_key(li)) * 16));
    s_acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(widen8(c[0], c[1]), qf.f[2 * j], s_acc, 0, 0, 0);
    s_acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(widen8(c[2], c[3]), qf.f[2 * j + 1], s_acc, 0, 0, 0);
  }
  return s_acc;
}

// O^T += V^T P^T from a tile of codes.  ds_read_b64_tr_b8: within 16 lanes, lane i receives byte i % 8 of the 8-byte vectors
// addressed by lanes i / 8, 2 + i / 8, .., 14 + i / 8 - one column of eight token rows, all an MFMA operand needs.  Lane k
// of a 16-lane group therefore addresses token row 16 u + 8 (t / 4) + 4 lh + t % 4, t = k / 2, bytes 8 (k % 2) .. of the
// group's 16 columns.
__device__ __forceinline__ void tile_pv8(const char* vbuf, const bf16x8_t pb2[2], SoftmaxState& st, int lane) {
  typedef __attribute__((ext_vector_type(2))) int i32x2_t;
  typedef __attribute__((address_space(3))) i32x2_t* lds_v2;
  const int lh = lane >> 5, k = lane & 15, t = k >> 1, g1 = (lane >> 4) & 1;
  const int row = 8 * (t >> 2) + 4 * lh + (t & 3);
  const int base = row * kAtRow8 + g1 * 16 + 8 * (k & 1);
  const int key = v8_key(row) * 16;
#pragma unroll
  for (int uu = 0; uu < 2; ++uu)
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      const i32x2_t c = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2)(vbuf + uu * 16 * kAtRow8 + base + ((32 * db) ^ key)));
      st.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(widen8(c[0], c[1]), pb2[uu], st.o[db], 0, 0, 0);
    }
}

// inclusive scan over the 64 lanes in six data-parallel additions: within each row of sixteen, then row 0 into 1 and row 2 into
// 3, then the lower half into the upper (every workgroup of a sweep waits for two of these before its first load)
__device__ __forceinline__ int wave_incl_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
  return x;
}

// A workgroup's share of a sweep: units u .. u_end - 1 (runs if by_run, else tiles), and the request b that holds the first one:
// L tokens long, units from .. to - 1 of the sweep.
struct Share { bool by_run; int u, u_end, b, L, from, to; };

// The lengths that a thread of build_split scans: its four requests'.  Asked for before anything else; what does not depend on
// them goes in between.
struct SplitLens { int n[4]; };
__device__ __forceinline__ SplitLens load_split_lens(const int32_t* __restrict__ seq_lens, int B) {
  const int t4 = threadIdx.x * 4;
  SplitLens r;
#pragma unroll
  for (int i = 0; i < 4; ++i) r.n[i] = t4 + i < B ? seq_lens[t4 + i] : 0;
  return r;
}

// The split of a sweep over few tokens, built by the whole workgroup (kThreads threads, B <= 1024).  If the pairs'
// tiles, cut into runs of kPar (one for each wavefront group that works at a time; a pair's last run may be shorter), are
// no more runs than there are workgroups (kWgs), a workgroup takes one run: s_pb[0 .. B] is the prefix of runs per request.
// Otherwise s_pb is the prefix of tiles, which are dealt out evenly (unit_begin).
// Runs of one pair each: a run that crosses from pair to pair pays a segment's fixed cost (query rows, first tiles, merge of the
// wavefronts: 3 to 4 us) for each in turn.  Shorter runs than kPar would leave wavefronts idle without ending any sooner, and
// every run adds a partial per query row to the merge.  32 query heads over 8 KV heads, five rows, us for sweep and merge with
// [tiles dealt out evenly to all workgroups; to as many as get kPar tiles each; one run each]: 1 request of 16 tokens 10.8, 21.8,
// 10.4; 8 of 64 tokens 11.8, 15.5, 11.4; 7 of 20 to 400 tokens 17.2, 22.8, 12.1; 4 of 1000 tokens 19.5, 14.7, 14.4.
// The thread whose request holds the workgroup's first unit says so: no search of the prefix, and no second trip for the length.
// A sweep's start is a chain of short trips (lengths, scan, first segment, query rows and page ids, tiles) in which no tile moves; with
// that, the query rows' divisions ahead of the scan and a later segment's length fetched under the one before it, us for the call:
// 16 trees of 32 over 4096 tokens 67.8 -> 66.2, 32 requests of five rows over 1024 to 4096 in fp8 40.7 -> 40.1, 64 of 100 to
// 600 tokens in bf16 32.0 -> 31.3, 8 of 64 to 128 10.6 -> 10.4; one request of 2777 tokens 11.9 -> 12.0, the backward within noise.
template <int kThreads, int kPar, int kWgs>
__device__ __forceinline__ Share build_split(const SplitLens& len, int B, int Hkv, int* s_pb, int2* s_wsum, int4* s_first) {
  const int t4 = threadIdx.x * 4, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int tiles[4], runs[4], nt = 0, nr = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int n = (len.n[i] + kAtTile - 1) / kAtTile;
    tiles[i] = n * Hkv;
    runs[i] = (n + kPar - 1) / kPar * Hkv;
    nt += tiles[i];
    nr += runs[i];
  }
  const int it = wave_incl_scan(nt), ir = wave_incl_scan(nr);
  if (lane == 63) s_wsum[wave] = make_int2(it, ir);
  __syncthreads();
  int at_tile = it - nt, at_run = ir - nr, all_tiles = 0, all_runs = 0;
#pragma unroll
  for (int w = 0; w < kThreads / kWave; ++w) {
    const int2 x = s_wsum[w];
    all_tiles += x.x;
    all_runs += x.y;
    at_tile += w < wave ? x.x : 0;
    at_run += w < wave ? x.y : 0;
  }
  all_tiles = __builtin_amdgcn_readfirstlane(all_tiles);
  all_runs = __builtin_amdgcn_readfirstlane(all_runs);
  Share r;
  r.by_run = all_runs <= kWgs;
  r.u = r.by_run ? (int)blockIdx.x : unit_begin(all_tiles, kWgs, blockIdx.x);
  r.u_end = r.by_run ? min(all_runs, r.u + 1) : unit_begin(all_tiles, kWgs, blockIdx.x + 1);
  r.b = r.L = r.from = r.to = 0;
  // Workgroups without a share end here (the first still publishes the split): where a launch has more of them than the chip holds
  // - several row blocks over a short context - the later blocks' working ones start behind them, and every wait that the idle ones
  // do not need is paid once a block.  One tree of 64 nodes, 48 query heads over 8 KV heads (three blocks), us for the call
  // with the idle ones held to the second barrier and now: 64 tokens 16.2, 15.4, 300 tokens 20.4, 19.4; 32 heads 14.5, 13.9.
  if (r.u >= r.u_end && blockIdx.x != 0) return r;
  int at = r.by_run ? at_run : at_tile;
  if (threadIdx.x == 0) s_pb[0] = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int from = at;
    at += r.by_run ? runs[i] : tiles[i];
    if (t4 + i < B) s_pb[t4 + i + 1] = at;
    if (r.u >= from && r.u < at) *s_first = make_int4(t4 + i, len.n[i], from, at);
  }
  __syncthreads();
  if (r.u < r.u_end) {
    const int4 f = *s_first;
    r.b = f.x;
    r.L = f.y;
    r.from = f.z;
    r.to = f.w;
  }
  return r;
}

// The same of the prefix of tiles that the planning kernel has left in memory.
template <int kWgs>
__device__ __forceinline__ Share load_split(const int32_t* __restrict__ PB, const int32_t* __restrict__ seq_lens, int B) {
  Share r;
  const int U = PB[B];
  r.by_run = false;
  r.u = unit_begin(U, kWgs, blockIdx.x);
  r.u_end = unit_begin(U, kWgs, blockIdx.x + 1);
  int lo = 0, hi = B - 1;  // largest b with PB[b] <= u
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (PB[mid] <= r.u) lo = mid; else hi = mid - 1;
  }
  r.b = lo;
  r.L = seq_lens[lo];
  r.from = PB[lo];
  r.to = PB[lo + 1];
  return r;
}

// The split for the merge kernel: the prefix of tiles as it is, the prefix of runs as complements (negative numbers).
__device__ __forceinline__ void publish_split(int32_t* __restrict__ PB, const int* s_pb, int B, bool by_run, int threads) {
  for (int i = threadIdx.x; i <= B; i += threads) PB[i] = by_run ? ~s_pb[i] : s_pb[i];
}

// The workgroups whose partials of the pair (b, hk), n_b tiles long, a merge kernel adds up: w0 .. w0 + np - 1 of the published
// split.  (A sequence of length 0 has no partial: np = 0.)
__device__ __forceinline__ void pair_owners(const int32_t* __restrict__ PB, int B, int b, int hk, int n_b, int wgs, int par,
                                            int& w0, int& np) {
  const int U = PB[B], first = PB[b];
  w0 = 0;
  np = 0;
  if (U < 0) {  // runs, one per workgroup
    np = (n_b + par - 1) / par;
    w0 = ~first + hk * np;
  } else if (n_b > 0) {
    w0 = unit_owner(U, wgs, first + hk * n_b);
    np = unit_owner(U, wgs, first + hk * n_b + n_b - 1) - w0 + 1;
  }
}

constexpr int kLocalPlanMax = 1024;  // up to this many requests every workgroup builds the prefix itself


}  // namespace aurora
