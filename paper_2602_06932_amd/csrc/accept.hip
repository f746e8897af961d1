// Acceptance walk and residual / bonus draw of the verification step (paper sections 2.1, 3.1,
// 3.3: the target keeps a prefix of the drafted chain - or a root-to-node path of the drafted
// tree - and emits one more token; accepted and rejected positions are both reported).
//
// Inputs are the fp32 logits written by the LM-head kernel and the per-(row, vocab tile) softmax
// statistics (max, sum exp, arg-max) of its epilogue.
//
// Chains at T > 0 (the serving default) take two small kernels so that the one vocabulary sweep a
// request needs is spread over the whole chip instead of one compute unit:
//   accept_chain_sweep  S workgroups per request.  Each repeats the cheap part - merge the tile
//                       statistics of the request's rows, evaluate the k accept tests
//                       u * q(d) < p(d) in parallel (fp64), find the first failure - and then sums
//                       the draw weights - max(0, p - q) after a rejection, p itself when every
//                       draft was kept - over groups of 256 tokens of its slice; slice 0 writes
//                       accept_len / accept_mask / p_at_draft / row_lse;
//   accept_chain_pick   one workgroup per request: scan the group sums, find the group holding
//                       u * total, rescan that group with a wavefront prefix sum for the token
//                       (done by the sweep's workgroup itself where S is 1).
// Trees at T > 0 may need one sweep per rejected sibling, each depending on the previous one:
// accept_tree_kernel walks a request in up to 16 workgroups that split every sweep and exchange their
// partial sums.  The same kernel, one workgroup per request, serves every greedy (T = 0) call, where no
// sweep exists.
// All sums are fp64 in a fixed order: results are reproducible bit for bit.
#include "common.hpp"
#include "launch.hpp"

#include <algorithm>

namespace aurora {

constexpr int kAccThreads = 1024;
constexpr int kAccWaves = kAccThreads / kWave;
constexpr int kMaxGroups = 4096;  // group sums kept in LDS by the tree kernel (32 KB of doubles): V <= 2^20
constexpr int kSmallThreads = 256;
constexpr int kSweepThreads = 512;  // chain sweep: eight wavefronts, so five rows merge and a 32-group slice sweeps in one round
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// Probability of token v at the current node after `nres` residual steps, in fp64 throughout (used
// for the accept tests).  p0 = exp(l / T - lse);  p_{s+1} = max(0, p_s - q) / Z_s.
__device__ __forceinline__ double node_weight(double p0, float qv, int nres, const double* Zs) {
  double x = p0;
  for (int s = 0; s < nres; ++s) x = fmax(0.0, x - (double)qv) / Zs[s];
  return x;
}

// The same quantity for the vocabulary sweeps.  The exponent is formed in fp64 (so the row's
// logsumexp enters unrounded), rounded once to fp32 and exponentiated by the hardware exp2, the
// function the LM-head epilogue used for the statistics lse was merged from - a bias of that
// function cancels between the two.  The fp32 rounding is an independent ~1e-7 relative
// perturbation per token and averages out of the running sums.  skip_last leaves the last residual
// step unnormalised (weights whose sum is Z_{nres-1}).  The normalisers enter as reciprocals: a
// multiplication per token and level instead of an fp64 division.
__device__ __forceinline__ double sweep_weight(float l, float qv, double lse, double inv_t, int nres,
                                               const double* invZs, bool skip_last) {
  const double a = ((double)l * inv_t - lse) * 1.4426950408889634;
  double x = (double)__builtin_amdgcn_exp2f((float)a);
  for (int s = 0; s < nres; ++s) {
    x = fmax(0.0, x - (double)qv);
    if (!(skip_last && s == nres - 1)) x *= invZs[s];
  }
  return x;
}

// Siblings drawn without replacement: the children of a node were drawn one after the other, each from the
// parent's q with the earlier siblings' tokens removed.  The draft distribution that residual level s was formed
// with is then q with the tokens rej[0 .. len[s]) set to zero, times fac[s] = 1 / (1 - their mass).
struct QLevels {
  const int* rej;
  const int* len;
  const double* fac;
};
__device__ __forceinline__ bool in_list(int v, const int* list, int n) {
  bool hit = false;
  for (int i = 0; i < n; ++i) hit |= list[i] == v;
  return hit;
}
__device__ __forceinline__ double node_weight_wor(double p0, float qv, int v, int nres, const double* Zs, const QLevels& ql) {
  double x = p0;
  for (int s = 0; s < nres; ++s) {
    const double qs = in_list(v, ql.rej, ql.len[s]) ? 0.0 : (double)qv * ql.fac[s];
    x = fmax(0.0, x - qs) / Zs[s];
  }
  return x;
}
__device__ __forceinline__ double sweep_weight_wor(float l, float qv, int v, double lse, double inv_t, int nres,
                                                   const double* invZs, bool skip_last, const QLevels& ql) {
  const double a = ((double)l * inv_t - lse) * 1.4426950408889634;
  double x = (double)__builtin_amdgcn_exp2f((float)a);
  for (int s = 0; s < nres; ++s) {
    const double qs = in_list(v, ql.rej, ql.len[s]) ? 0.0 : (double)qv * ql.fac[s];
    x = fmax(0.0, x - qs);
    if (!(skip_last && s == nres - 1)) x *= invZs[s];
  }
  return x;
}

__device__ __forceinline__ double wave_incl_scan(double x, int lane) {
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const double y = __shfl_up(x, o, kWave);
    if (lane >= o) x += y;
  }
  return x;
}

struct AcceptParams {
  int Nq, V, n_tiles, slices, gmul, ngroups;
  float temperature;
  const float* logits;
  float* pmax;
  float* psum;
  int32_t* parg;
  const int32_t* tok;
  const float* q;       // draft probabilities, row stride Vq
  const int32_t* t2d;   // target id -> index into a row of q, or -1 (q = 0 there); NULL: q rows are dense over V
  int Vq;               // entries per row of q: the draft vocabulary, or V
  const float* un;
  const int32_t* parents;
  int32_t* accept_len;
  int32_t* next_token;
  uint8_t* accept_mask;
  float* p_at_draft;
  float* row_lse;
  // scratch of the chain path
  double* st_lse;     // [B] logsumexp of the row the draw happens on
  int32_t* st_row;    // [B] that row (= accept_len)
  int32_t* st_rej;    // [B] 1: draw from max(0, p - q); 0: draw from p
  double* gsum;       // [B, ngroups]
  int32_t* lastpos;   // [B, slices] largest token with positive weight per slice, or -1
  // tree path with several workgroups per request: [B, 2, 2, tree_slices] halves of the slices' sums, zeros at launch
  unsigned long long* exch;
  const float* temps;  // [B] one temperature per request (0 = that request is verified greedily), or NULL
  int wor;             // tree walk: siblings were drawn without replacement
  int solo_slices;     // tree walk with one workgroup: slices it sweeps the vocabulary in
  int spin_limit;      // tree walk with several workgroups: polls of the others' sums before giving up
};

// the temperature of request b: its own, or the call's
__device__ __forceinline__ float request_temperature(const AcceptParams& P, int b) {
  return P.temps ? P.temps[b] : P.temperature;
}

// (max, logsumexp(l / T), arg-max) of one logits row, merged from its tile statistics by one
// wavefront; result valid in every lane.  The row's maximum first, over the lanes, then the sums scaled to it: no running
// rescale, so no chain of exponentials.  All of a row's statistics are in flight together and stay in registers up to
// kHeldTiles of them; the later ones of a larger vocabulary are read twice.  Scale factors go through the hardware exp2 of an
// fp64-formed exponent.
constexpr int kHeldTiles = 832;  // 212 992 vocabulary entries
__device__ __forceinline__ void merge_row_stats(const AcceptParams& P, size_t row, double T, int lane, float* out_max,
                                                double* out_lse, int* out_arg, bool want_arg = true) {
  constexpr int kHeld = kHeldTiles / kWave;
  const int nt = P.n_tiles;
  const float* pm = P.pmax + row * nt;
  const float* ps = P.psum + row * nt;
  const double c = 1.4426950408889634 / T;
  float xm[kHeld], xs[kHeld];
#pragma unroll
  for (int u = 0; u < kHeld; ++u) {
    xm[u] = -INFINITY;
    xs[u] = 0.f;
    if (u * kWave < nt) {  // uniform
      const int t = u * kWave + lane, tc = t < nt ? t : nt - 1;
      xm[u] = pm[tc];
      xs[u] = t < nt ? ps[tc] : 0.f;
    }
  }
  float m = -INFINITY;
#pragma unroll
  for (int u = 0; u < kHeld; ++u) m = fmaxf(m, xm[u]);  // (past the end: the last tile once more)
  for (int t = kHeldTiles + lane; t < nt; t += kWave) m = fmaxf(m, pm[t]);
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, kWave));
  const double md = m > -INFINITY ? (double)m : 0.0;
  double s = 0.0;
  int mt = 0x7fffffff;
#pragma unroll
  for (int u = kHeld - 1; u >= 0; --u)
    if (u * kWave < nt) {
      // (a tile of -inf alone has no sum; whatever stands in its place is not read into s)
      s += xm[u] > -INFINITY ? (double)xs[u] * (double)__builtin_amdgcn_exp2f((float)(((double)xm[u] - md) * c)) : 0.0;
      if (xm[u] == m) mt = min(u * kWave + lane, nt - 1);
    }
  for (int t = kHeldTiles + lane; t < nt; t += kWave) {
    const float x = pm[t];
    if (x > -INFINITY) s += (double)ps[t] * (double)__builtin_amdgcn_exp2f((float)(((double)x - md) * c));
    if (x == m) mt = min(mt, t);
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, kWave);
  *out_max = m;
  *out_lse = (double)m / T + log(s);
  *out_arg = 0;
  if (want_arg) {
    // the arg-max id (lowest tile that holds the maximum) sits behind one more dependent load; only greedy verification reads it
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) mt = min(mt, __shfl_xor(mt, o, kWave));
    *out_arg = P.parg[row * nt + (mt < nt ? mt : 0)];
  }
}

// The sum over a row of sixteen lanes, in every one of them, added over distances of 8, 4, 2 and 1 lanes (after each turn by that
// distance the values repeat with it, so turning the row is exchanging).
__device__ __forceinline__ float row16_sum(float x) {
  x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x128, 0xf, 0xf, false));
  x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x124, 0xf, 0xf, false));
  x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x122, 0xf, 0xf, false));
  x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x121, 0xf, 0xf, false));
  return x;
}

// The same from the logits themselves, where no kernel has formed the tile statistics (generic LM head, small vocabulary), which
// are left behind as row_tile_stats leaves them, bit for bit: per tile the maximum, its lowest index and the sum of
// exp((l - max) / T) in that kernel's order.  Its thread t adds the entries t, t + 256, .. of a tile, its wavefronts add over
// distances of 32, 16, .. 1 threads, and their four sums are added in turn.  Here element e of lane l's four vectors is thread
// 4 l + e: a wavefront there is a row of sixteen lanes here, its distances of 32 to 4 are 8 to 1 lanes, the last two are elements.
constexpr int kRowStatTiles = 2;
__device__ __forceinline__ void form_row_stats(const AcceptParams& P, size_t row, double T, int lane, float* out_max,
                                               double* out_lse, int* out_arg) {
  const int V = P.V, nt = P.n_tiles;
  const float* lr = P.logits + row * V;
  const float inv_t = 1.f / (float)T;
  const bool vec = (V & 3) == 0;
  float tile_m = -INFINITY, tile_s = 0.f;  // lane t: those of tile t
  int tile_arg = 0x7fffffff;
#pragma unroll 1
  for (int t = 0; t < nt; ++t) {
    float x[16];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int v = t * kRowStatTile + c * 256 + lane * 4;
      if (vec && v < V) {
        const f32x4_t y = *(const f32x4_t*)(lr + v);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * c + e] = y[e];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * c + e] = v + e < V ? lr[v + e] : -INFINITY;
      }
    }
    float mx = -INFINITY;  // (a NaN is no maximum)
#pragma unroll
    for (int i = 0; i < 16; ++i) mx = fmaxf(mx, x[i]);
    mx = wave_max(mx);
    // what lies past the vocabulary is told by its index: a NaN has to reach the sum, and with it the row's logsumexp
    int at = 0x7fffffff;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int v = t * kRowStatTile + (i >> 2) * 256 + lane * 4 + (i & 3);
      s[i & 3] += v < V ? __expf((x[i] - mx) * inv_t) : 0.f;
    }
#pragma unroll
    for (int i = 15; i >= 0; --i) {
      const int v = t * kRowStatTile + (i >> 2) * 256 + lane * 4 + (i & 3);
      at = x[i] > -INFINITY && x[i] == mx ? v : at;
    }
    // the lowest index: of the first of the tile's quarters that holds one, the first lane's
    unsigned long long hit = 0;
#pragma unroll
    for (int c = 3; c >= 0; --c) {
      const unsigned long long here = __ballot(((at - t * kRowStatTile) >> 8) == c);
      hit = here ? here : hit;
    }
    at = __builtin_amdgcn_readlane(at, hit ? __ffsll((long long)hit) - 1 : 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = row16_sum(s[e]);
    const unsigned row_s = __float_as_uint((s[0] + s[2]) + (s[1] + s[3]));
    float sum = __uint_as_float(__builtin_amdgcn_readlane(row_s, 0));
#pragma unroll
    for (int r = 1; r < 4; ++r) sum += __uint_as_float(__builtin_amdgcn_readlane(row_s, 16 * r));
    if (lane == t) {
      tile_m = mx;
      tile_s = sum;
      tile_arg = at;
    }
  }
  if (lane < nt) {
    P.pmax[row * nt + lane] = tile_m;
    P.psum[row * nt + lane] = tile_s;
    P.parg[row * nt + lane] = tile_arg;
  }
  const float m = wave_max(tile_m);
  const double md = m > -INFINITY ? (double)m : 0.0, c = 1.4426950408889634 / T;
  const double s = wave_sum(tile_m > -INFINITY ? (double)tile_s * (double)__builtin_amdgcn_exp2f((float)(((double)tile_m - md) * c)) : 0.0);
  *out_max = m;
  *out_lse = (double)m / T + log(s);
  *out_arg = wave_min(tile_m == m ? tile_arg : 0x7fffffff);
}

// ============================================================================================
// Chain path.  A group is 256 consecutive tokens: lane i of the wavefront that owns it holds tokens
// 4i .. 4i+3 (one 16-byte load per row when the row is 16-byte aligned).
// ============================================================================================
constexpr int kGroup = 256;

// the logits and draft probabilities of the four tokens v0 .. v0+3 a lane owns
struct Lane4 { float l[4], q[4]; };
// One row of draft probabilities: dense over the target vocabulary, or compact over the draft vocabulary
// with the target -> draft index map (entries off the draft vocabulary have probability 0).
struct QRow {
  const float* row;
  const int32_t* t2d;
};
// 16-byte loads of the logits row and of the q row (or of the index map) are possible
__device__ __forceinline__ bool rows_vec_ok(const AcceptParams& P) {
  const uintptr_t qa = P.t2d ? (uintptr_t)P.t2d : (uintptr_t)P.q;
  return (P.V & 3) == 0 && ((qa | (uintptr_t)P.logits) & 15) == 0;
}
__device__ __forceinline__ QRow q_row(const AcceptParams& P, size_t r) { return QRow{P.q + r * (size_t)P.Vq, P.t2d}; }
__device__ __forceinline__ float q_at(const QRow& q, int v) {
  if (!q.t2d) return q.row[v];
  const int j = q.t2d[v];
  return j >= 0 ? q.row[j] : 0.f;
}
typedef __attribute__((ext_vector_type(4))) int i32x4_t;
__device__ __forceinline__ Lane4 lane_load(const float* __restrict__ lrow, const QRow& q, int v0, int V, bool vec_ok) {
  Lane4 r;
  if (vec_ok && v0 + 3 < V) {
    const f32x4_t lv = *(const f32x4_t*)(lrow + v0);
#pragma unroll
    for (int e = 0; e < 4; ++e) r.l[e] = lv[e];
    if (!q.t2d) {
      const f32x4_t qv = *(const f32x4_t*)(q.row + v0);
#pragma unroll
      for (int e = 0; e < 4; ++e) r.q[e] = qv[e];
    } else {
      const i32x4_t jv = *(const i32x4_t*)(q.t2d + v0);
#pragma unroll
      for (int e = 0; e < 4; ++e) r.q[e] = jv[e] >= 0 ? q.row[jv[e]] : 0.f;
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      r.l[e] = v0 + e < V ? lrow[v0 + e] : -INFINITY;
      r.q[e] = v0 + e < V ? q_at(q, v0 + e) : 0.f;
    }
  }
  return r;
}
// their draw weights (0 past the end of the vocabulary)
__device__ __forceinline__ void lane_weights(const Lane4& r, int v0, int V, double lse, double inv_t, int nres,
                                             double x[4], const double* invZs = nullptr, bool skip_last = true) {
#pragma unroll
  for (int e = 0; e < 4; ++e)
    x[e] = v0 + e < V ? sweep_weight(r.l[e], r.q[e], lse, inv_t, nres, invZs, skip_last) : 0.0;
}

__device__ __forceinline__ void lane_weights_wor(const Lane4& r, int v0, int V, double lse, double inv_t, int nres,
                                                 double x[4], const double* invZs, bool skip_last, const QLevels& ql) {
#pragma unroll
  for (int e = 0; e < 4; ++e)
    x[e] = v0 + e < V ? sweep_weight_wor(r.l[e], r.q[e], v0 + e, lse, inv_t, nres, invZs, skip_last, ql) : 0.0;
}

// Inverse-CDF draw from the group sums of one request by a workgroup of kThreads: the stop row, whether the draw is from the
// residual (nres = 1) or from p, and the row's logsumexp are the sweep's.
// A residual that vanished (sum 0) falls back to the row's p: rare enough for one workgroup.
template <int kThreads>
__device__ __forceinline__ void chain_pick(const AcceptParams& P, int b, int row, int nres, double lse) {
  __shared__ double s_wtot[kThreads / kWave];
  __shared__ int s_pick;
  __shared__ double s_prefix;
  const int tid = threadIdx.x, lane = tid % kWave, wv = tid / kWave;
  const int V = P.V, ng = P.ngroups;
  const double inv_t = 1.0 / (double)request_temperature(P, b);
  const float* lrow = P.logits + ((size_t)b * P.Nq + row) * V;
  const QRow qrow = q_row(P, (size_t)b * P.Nq + row);
  const bool vec_ok = rows_vec_ok(P);
  double* gs = P.gsum + (size_t)b * ng;
  const int per = (ng + kThreads - 1) / kThreads;
  const int ga = min(ng, tid * per), gb = min(ng, ga + per);

  for (int attempt = 0; attempt < 2; ++attempt) {
    double loc = 0.0;
    for (int g = ga; g < gb; ++g) loc += gs[g];
    const double incl = wave_incl_scan(loc, lane);
    if (lane == kWave - 1) s_wtot[wv] = incl;
    if (tid == 0) s_pick = 0x7fffffff;
    __syncthreads();
    double wbase = 0.0, total = 0.0;
    for (int i = 0; i < kThreads / kWave; ++i) {
      if (i < wv) wbase += s_wtot[i];
      total += s_wtot[i];
    }
    if (total > 0.0 || nres == 0) {
      const double thr = (double)P.un[((size_t)b * P.Nq + row) * 2 + 1] * total;
      double run = wbase + incl - loc;
      int found = 0x7fffffff;
      double before = 0.0;
      for (int g = ga; g < gb; ++g) {
        const double nxt = run + gs[g];
        if (found == 0x7fffffff && nxt > thr) { found = g; before = run; }
        run = nxt;
      }
      if (found != 0x7fffffff) atomicMin(&s_pick, found);
      __syncthreads();
      const int pick = s_pick;
      if (pick == found && found != 0x7fffffff) s_prefix = before;
      __syncthreads();
      if (wv == 0) {
        int token = -1;
        if (pick != 0x7fffffff) {
          const int v0 = pick * kGroup + lane * 4;
          double x[4];
          lane_weights(lane_load(lrow, qrow, v0, V, vec_ok), v0, V, lse, inv_t, nres, x);
          const double lane_tot = (x[0] + x[1]) + (x[2] + x[3]);
          const double lane_incl = wave_incl_scan(lane_tot, lane) + s_prefix;
          const unsigned long long hit = __ballot(lane_incl > thr);
          const unsigned long long pos = __ballot(lane_tot > 0.0);
          if (hit) {
            const int hl = __ffsll((long long)hit) - 1;  // first lane whose running sum crosses
            double r0 = __shfl(lane_incl - lane_tot, hl, kWave);
            int e_hit = 3;
            const double y0 = __shfl(x[0], hl, kWave), y1 = __shfl(x[1], hl, kWave), y2 = __shfl(x[2], hl, kWave);
            if (r0 + y0 > thr) e_hit = 0;
            else if (r0 + y0 + y1 > thr) e_hit = 1;
            else if (r0 + y0 + y1 + y2 > thr) e_hit = 2;
            token = pick * kGroup + hl * 4 + e_hit;
            if (token >= V) token = -1;
          } else if (pos) {
            // rounding left no crossing inside the group: its last token with positive weight
            const int pl = 63 - __clzll((long long)pos);
            int e_last = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (__shfl(x[e], pl, kWave) > 0.0) e_last = e;
            token = pick * kGroup + pl * 4 + e_last;
          }
        }
        if (token < 0) {  // no crossing at all: the largest token with positive weight
          int m = -1;
          for (int i = lane; i < P.slices; i += kWave) m = max(m, P.lastpos[(size_t)b * P.slices + i]);
          token = wave_max(m);
        }
        if (lane == 0) P.next_token[b] = token;
      }
      return;
    }
    // residual identically zero: recompute the group sums of p itself with this workgroup, then draw
    __syncthreads();
    nres = 0;
    int lastpos = -1;
    for (int g = wv; g < ng; g += kThreads / kWave) {
      const int v0 = g * kGroup + lane * 4;
      double x[4];
      lane_weights(lane_load(lrow, qrow, v0, V, vec_ok), v0, V, lse, inv_t, 0, x);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (x[e] > 0.0) lastpos = max(lastpos, v0 + e);
      const double acc = wave_sum((x[0] + x[1]) + (x[2] + x[3]));
      if (lane == 0) gs[g] = acc;
    }
    lastpos = wave_max(lastpos);
    if (lane == 0) atomicMax(&P.lastpos[(size_t)b * P.slices], lastpos);
    __threadfence_block();
    __syncthreads();
  }
}

// Kernel 1: S workgroups per request.  Every workgroup repeats the (cheap) walk - merge the tile
// statistics of the request's rows, evaluate the k accept tests in parallel in fp64, find the first
// failure - then sums the draw weights over its slice of the vocabulary.  Slice 0 writes the
// per-request outputs and the state the draw kernel needs.
// kForm: the tile statistics are formed here too.
template <bool kForm>
__global__ __launch_bounds__(kSweepThreads) void accept_chain_sweep(AcceptParams P) {
  __shared__ double s_lse[kMaxNq];
  __shared__ int s_ok[kMaxNq], s_arg[kMaxNq];
  __shared__ int s_last[kSweepThreads / kWave];
  const int slice = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid % kWave, wv = tid / kWave;
  const int Nq = P.Nq, V = P.V;
  // with one temperature per request, a request at T = 0 is verified greedily inside this kernel
  const float Tf = request_temperature(P, b);
  const bool greedy = !(Tf > 0.f);
  const double T = greedy ? 1.0 : (double)Tf;
  const size_t row0 = (size_t)b * Nq;
  // operands of the accept tests: their addresses are known up front, so the loads fly during the merge
  float t_l = 0.f, t_q = 0.f, t_u = 0.f;
  int t_tok = -1;
  if (tid > 0 && tid < Nq) {
    t_tok = P.tok[row0 + tid];
    t_l = P.logits[(row0 + tid - 1) * V + t_tok];
    t_q = q_at(q_row(P, row0 + tid - 1), t_tok);
    t_u = P.un[(row0 + tid) * 2 + 0];
  }
  for (int n = wv; n < Nq; n += kSweepThreads / kWave) {
    float mx; double lse; int arg;
    if constexpr (kForm) form_row_stats(P, row0 + n, T, lane, &mx, &lse, &arg);
    else merge_row_stats(P, row0 + n, T, lane, &mx, &lse, &arg, greedy);
    if (lane == 0) { s_lse[n] = lse; s_arg[n] = arg; }
  }
  __syncthreads();
  if (tid < Nq) {
    const int n = tid;
    float pv = 0.f;
    int ok = 1;
    if (n > 0 && greedy) {
      ok = t_tok == s_arg[n - 1];
      pv = ok ? 1.f : 0.f;
    } else if (n > 0) {
      const double p = exp((double)t_l / T - s_lse[n - 1]);
      ok = ((double)t_u * (double)t_q < p) ? 1 : 0;
      pv = (float)p;
    }
    s_ok[n] = ok;
    if (slice == 0) {
      if (P.p_at_draft) P.p_at_draft[row0 + n] = pv;
      if (P.row_lse) P.row_lse[row0 + n] = (float)s_lse[n];
    }
  }
  __syncthreads();
  int first_fail = Nq;
  for (int n = 1; n < Nq; ++n)
    if (!s_ok[n]) { first_fail = n; break; }
  const int row = first_fail - 1;          // accepted drafts = index of the row the draw happens on
  const int nres = first_fail < Nq ? 1 : 0;  // 1: draw from max(0, p - q); 0: all kept, draw from p
  const double lse = s_lse[row];
  if (slice == 0) {
    if (tid < Nq) P.accept_mask[row0 + tid] = tid <= row ? 1 : 0;
    if (tid == 0) {
      P.accept_len[b] = row;
      P.st_row[b] = row;
      P.st_rej[b] = greedy ? 2 : nres;  // 2: nothing left for the draw kernel
      P.st_lse[b] = lse;
      if (greedy) P.next_token[b] = s_arg[row];
    }
  }
  if (greedy) return;  // the whole workgroup: a greedy request has no sweep

  const double inv_t = 1.0 / T;
  const float* lrow = P.logits + (row0 + row) * V;
  const QRow qrow = q_row(P, row0 + row);
  const bool vec_ok = rows_vec_ok(P);
  const int per = (P.ngroups + P.slices - 1) / P.slices;
  const int g0 = slice * per, g1 = min(P.ngroups, g0 + per);
  int lastpos = -1;
  constexpr int kBatch = 4;  // groups whose loads a wavefront keeps in flight together
  constexpr int kStep = kSweepThreads / kWave;
  for (int g = g0 + wv; g < g1; g += kBatch * kStep) {
    Lane4 r[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int gi = g + i * kStep;
      if (gi < g1) r[i] = lane_load(lrow, qrow, gi * kGroup + lane * 4, V, vec_ok);
    }
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int gi = g + i * kStep;
      if (gi < g1) {  // wave-uniform
        const int v0 = gi * kGroup + lane * 4;
        double x[4];
        lane_weights(r[i], v0, V, lse, inv_t, nres, x);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (x[e] > 0.0) lastpos = max(lastpos, v0 + e);
        const double sg = wave_sum((x[0] + x[1]) + (x[2] + x[3]));
        if (lane == 0) P.gsum[(size_t)b * P.ngroups + gi] = sg;
      }
    }
  }
  lastpos = wave_max(lastpos);
  if (lane == 0) s_last[wv] = lastpos;
  __syncthreads();
  if (tid == 0) {
    int m = -1;
    for (int i = 0; i < kSweepThreads / kWave; ++i) m = max(m, s_last[i]);
    P.lastpos[(size_t)b * P.slices + slice] = m;
  }
  // one slice (small vocabularies, or batches that fill the chip): the draw follows here instead of behind another launch
  if (P.slices == 1) {
    __threadfence_block();
    __syncthreads();
    chain_pick<kSweepThreads>(P, b, row, nres, lse);
  }
}

// Kernel 2: the draw for requests whose sweep was spread over several workgroups.
__global__ __launch_bounds__(kSmallThreads) void accept_chain_pick(AcceptParams P) {
  const int b = blockIdx.x;
  const int nres = P.st_rej[b];
  if (nres == 2) return;  // a greedy request (one temperature per request): its token is already written
  chain_pick<kSmallThreads>(P, b, P.st_row[b], nres, P.st_lse[b]);
}

// ============================================================================================
// Trees at T > 0, and every greedy call.  Grid (S, B): S workgroups per request, each sweeping one slice of the vocabulary.
// Every workgroup repeats the walk (the same inputs give the same decisions, bit for bit); a sweep's slice sums are
// exchanged through global memory and added in slice order by all.  The final draw is made by the workgroup whose slice
// holds the crossing.
//
// The walk is a chain of dependent sweeps (a rejected sibling's residual needs the normaliser of the level before), so what
// counts is the time from one exchange to the next.  A sweep at the node of the previous one finds its logits and draft
// probabilities in registers; a rejection needs only the slice's total (group sums are formed for the draw alone); the walk's
// state lives in registers of every wavefront - the tree is a lane per node, the next child a ballot - so a step has two
// workgroup barriers; and a slice sum is its own flag: it travels as two words, each half of the sum beside the number of the
// sweep, so one store and one load cross the dies and nothing is ordered against anything else.  The words of two sweeps in
// turn are enough: a workgroup that stores for sweep k + 2 has seen everybody's words of k + 1, which are stored once those of k
// have been read.  16 trees of 32 nodes over 128 256 ids: 90 us with group sums exchanged behind an arrival counter
// (release, acquire, then the loads; the rows re-read for every sweep) -> 39 us.
// The launcher keeps S * B within the number of compute units, so all workgroups of a request are resident together;
// the wait is bounded all the same.
// ============================================================================================
constexpr int kTreeMaxSlices = 16;
constexpr int kSpinLimit = 1 << 15;  // default number of polls (tens of milliseconds) before a workgroup stops waiting

// What a workgroup reads from another are 64-bit words, written and read with device-scope atomic accesses that go past the
// die-local caches.
__device__ __forceinline__ void store_word(unsigned long long* p, unsigned long long u) {
  __hip_atomic_store(p, u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long load_word(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int lane_value(int x, int lane) { return __builtin_amdgcn_readlane(x, lane); }
__device__ __forceinline__ float lane_value(float x, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
}
__device__ __forceinline__ double lane_value(double x, int lane) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(u & 0xffffffffu), lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(u >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// kHeld: a slice has at most held_groups(kWor) groups per wavefront, whose operands stay in registers from sweep to sweep (as
// many as 128 registers a thread take without spilling).  kWor: siblings were drawn without replacement.
__host__ __device__ constexpr int held_groups(bool wor) { return wor ? 2 : 3; }
#define AURORA_INLINE __attribute__((always_inline))
template <bool kHeld, bool kWor>
__global__ __launch_bounds__(kAccThreads) void accept_tree_kernel(AcceptParams P) {
  __shared__ double s_lse[kMaxNq];
  __shared__ int s_arg[kMaxNq];
  __shared__ double s_gsum[kMaxGroups];
  __shared__ double s_wtot[kAccWaves], s_tot[kTreeMaxSlices];
  __shared__ double s_share[kTreeMaxSlices][kAccWaves];  // the wavefronts' shares of the slices' totals
  __shared__ int s_fail, s_pick, s_lastpos;
  __shared__ double s_pick_prefix;
  __shared__ int s_par[kMaxNq], s_tok[kMaxNq];
  __shared__ float s_u0[kMaxNq], s_u1[kMaxNq];
  __shared__ float s_qtok[kMaxNq];  // draft probability of node n's token in its parent's row
  __shared__ double s_p0[kMaxNq];   // target probability of node n's token in its parent's row
  // Residual levels of the current node, one copy per wavefront (no barrier orders one wavefront's next step against
  // another's): normalisers; and, for siblings drawn without replacement, the tokens rejected here and the draft
  // distribution each level was formed with (see QLevels).
  __shared__ double s_Zw[kAccWaves][kMaxNq], s_invZw[kAccWaves][kMaxNq], s_qfacw[kAccWaves][kMaxNq];
  __shared__ int s_rejw[kAccWaves][kMaxNq], s_qlenw[kAccWaves][kMaxNq];

  const int b = blockIdx.y;
  // slices of the vocabulary: one per workgroup, or those that the request's only workgroup sweeps one after the other
  const bool alone = gridDim.x == 1;
  const int S = alone ? P.solo_slices : (int)gridDim.x, slice = blockIdx.x;
  const bool writer = slice == 0;                     // the workgroup that stores the walk's outputs
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int Nq = P.Nq, V = P.V;
  const float Tf = request_temperature(P, b);
  const bool greedy = !(Tf > 0.f);
  const double T = greedy ? 1.0 : (double)Tf;
  const double inv_t = 1.0 / T;
  const size_t row0 = (size_t)b * Nq;
  // operands of the accept tests: their addresses do not depend on the statistics, so the loads fly during the merge
  int t_par = -1, t_tok = 0;
  float t_l = 0.f, t_q = 0.f;
  if (tid < Nq) {
    t_par = P.parents ? P.parents[row0 + tid] : tid - 1;
    t_tok = P.tok[row0 + tid];
    s_par[tid] = t_par;
    s_tok[tid] = t_tok;
    s_u0[tid] = greedy ? 0.f : P.un[(row0 + tid) * 2 + 0];
    s_u1[tid] = greedy ? 0.f : P.un[(row0 + tid) * 2 + 1];
    if (tid > 0 && !greedy) {
      t_l = P.logits[(row0 + t_par) * V + t_tok];
      t_q = q_at(q_row(P, row0 + t_par), t_tok);
    }
  }

  // ---- 1. per-row (logsumexp, arg-max) from the tile statistics ---------------------------------
  for (int n = wv; n < Nq; n += kAccWaves) {
    float mx; double lse; int arg;
    merge_row_stats(P, row0 + n, T, lane, &mx, &lse, &arg, greedy);
    if (lane == 0) { s_lse[n] = lse; s_arg[n] = arg; }
  }
  if (tid == 0) s_fail = 0;
  __syncthreads();

  // ---- per-node outputs ------------------------------------------------------------------------
  if (tid < Nq) {
    const int n = tid;
    if (P.row_lse && writer) P.row_lse[row0 + n] = (float)s_lse[n];
    float pv = 0.f;
    if (n > 0) {
      if (greedy) {
        pv = (t_tok == s_arg[t_par]) ? 1.f : 0.f;
      } else {
        const double p0 = exp((double)t_l / T - s_lse[t_par]);
        s_p0[n] = p0;
        s_qtok[n] = t_q;
        pv = (float)p0;
      }
    }
    if (writer) {
      if (P.p_at_draft) P.p_at_draft[row0 + n] = pv;
      P.accept_mask[row0 + n] = n == 0 ? 1 : 0;
    }
  }
  __syncthreads();

  // ---- 2a. greedy walk: thread 0 only -----------------------------------------------------------
  if (greedy) {
    if (tid == 0 && writer) {
      int cur = 0, depth = 0;
      for (;;) {
        int moved = 0;
        for (int c = cur + 1; c < Nq && !moved; ++c) {
          if (s_par[c] == cur && s_tok[c] == s_arg[cur]) {
            cur = c;
            ++depth;
            P.accept_mask[row0 + c] = 1;
            moved = 1;
          }
        }
        if (!moved) break;
      }
      P.accept_len[b] = depth;
      P.next_token[b] = s_arg[cur];
    }
    return;
  }

  // ---- 2b. sampling walk: every wavefront for itself, meeting in the sweeps ----------------------
  // lane n of every wavefront holds node n
  const bool node = lane < Nq;
  const int n_par = node ? s_par[lane] : -2, n_tok = node ? s_tok[lane] : 0;
  const float n_u0 = node ? s_u0[lane] : 0.f, n_q = node && lane > 0 ? s_qtok[lane] : 0.f;
  const double n_p0 = node && lane > 0 ? s_p0[lane] : 0.0;
  double *Zs = s_Zw[wv], *invZs = s_invZw[wv], *qfac = s_qfacw[wv];
  int *rej = s_rejw[wv], *qlen = s_qlenw[wv];

  const int ngroups = (V + kGroup - 1) / kGroup;  // <= kMaxGroups (checked by the launcher)
  const bool vec_ok = rows_vec_ok(P);
  const int per_slice = (ngroups + S - 1) / S;
  auto slice_lo = [&](int s) AURORA_INLINE { return min(ngroups, s * per_slice); };
  bool solo = alone;  // this workgroup sweeps every slice itself
  const QLevels ql = {rej, qlen, qfac};

  int cur = 0, depth = 0, last_child = 0, nres = 0, sweeps = 0;
  bool have_total = false;  // `total` and s_tot are those of the current node's weights
  double total = 0.0;
  int cur_len = 0;          // siblings without replacement: the distribution the next sibling was drawn from
  double cur_fac = 1.0, rej_mass = 0.0;
  constexpr int kHold = kHeld ? held_groups(kWor) : 4;  // groups of a wavefront at a time
  // Held operands: the weights of residual level held_level and the draft probabilities of this lane's tokens.
  double held_x[kHeld ? kHold : 1][4];
  float held_q[kHeld ? kHold : 1][4];
  int held_node = -1, held_slice = -1, held_level = 0;

  // the weights (of residual level `level`; skip_last leaves its last step unnormalised) of the four tokens v0 ..
  auto weights = [&](const Lane4& r, int v0, int level, bool skip_last, double x[4]) AURORA_INLINE {
    if constexpr (kWor) lane_weights_wor(r, v0, V, s_lse[cur], inv_t, level, x, invZs, skip_last, ql);
    else lane_weights(r, v0, V, s_lse[cur], inv_t, level, x, invZs, skip_last);
  };
  // one residual step from level s, as the functions above take it: max(0, x - q), not yet normalised
  auto step = [&](double x, float q, int v, int s) AURORA_INLINE -> double {
    if constexpr (kWor) return fmax(0.0, x - (in_list(v, rej, qlen[s]) ? 0.0 : (double)q * qfac[s]));
    return fmax(0.0, x - (double)q);
  };
  // f(group, its weights in this lane's four tokens) for this wavefront's groups of slice sl, in ascending order
  auto for_groups = [&](int sl, int level, bool skip_last, auto f) AURORA_INLINE {
    const int lo = slice_lo(sl), hi = slice_lo(sl + 1);
    const float* lrow = P.logits + (row0 + cur) * V;
    const QRow qrow = q_row(P, row0 + cur);
    if constexpr (kHeld) {
      if (held_node != cur || held_slice != sl) {
        Lane4 r[kHold];
#pragma unroll
        for (int i = 0; i < kHold; ++i) {
          const int gi = lo + wv + i * kAccWaves;
          if (gi < hi) r[i] = lane_load(lrow, qrow, gi * kGroup + lane * 4, V, vec_ok);
        }
#pragma unroll
        for (int i = 0; i < kHold; ++i) {
          const int gi = lo + wv + i * kAccWaves;
          if (gi < hi) {
            weights(r[i], gi * kGroup + lane * 4, 0, false, held_x[i]);
#pragma unroll
            for (int e = 0; e < 4; ++e) held_q[i][e] = r[i].q[e];
          }
          __builtin_amdgcn_sched_barrier(0);  // a group at a time: the registers hold the operands
        }
        held_node = cur;
        held_slice = sl;
        held_level = 0;
      }
      for (; held_level < (skip_last ? level - 1 : level); ++held_level) {
        const double iz = invZs[held_level];
#pragma unroll
        for (int i = 0; i < kHold; ++i) {
          const int gi = lo + wv + i * kAccWaves;
          if (gi < hi)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              held_x[i][e] = step(held_x[i][e], held_q[i][e], gi * kGroup + lane * 4 + e, held_level) * iz;
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int i = 0; i < kHold; ++i) {
        const int gi = lo + wv + i * kAccWaves;
        if (gi < hi) {  // wave-uniform
          double x[4];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            x[e] = skip_last ? step(held_x[i][e], held_q[i][e], gi * kGroup + lane * 4 + e, held_level) : held_x[i][e];
          f(gi, x);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      for (int g = lo + wv; g < hi; g += kHold * kAccWaves) {
        Lane4 r[kHold];
#pragma unroll
        for (int i = 0; i < kHold; ++i) {
          const int gi = g + i * kAccWaves;
          if (gi < hi) r[i] = lane_load(lrow, qrow, gi * kGroup + lane * 4, V, vec_ok);
        }
#pragma unroll
        for (int i = 0; i < kHold; ++i) {
          const int gi = g + i * kAccWaves;
          if (gi < hi) {
            double x[4];
            weights(r[i], gi * kGroup + lane * 4, level, skip_last, x);
            f(gi, x);
          }
        }
      }
    }
  };
  // this wavefront's share of a slice's total, parked for the workgroup
  auto park_share = [&](int sl, int level, bool skip_last) AURORA_INLINE {
    double acc = 0.0;
    for_groups(sl, level, skip_last, [&](int, const double* x) AURORA_INLINE { acc += (x[0] + x[1]) + (x[2] + x[3]); });
    acc = wave_sum(acc);
    if (lane == 0) s_share[sl][wv] = acc;
  };
  auto slice_sum = [&](int sl) AURORA_INLINE {
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < kAccWaves; ++i) t += s_share[sl][i];
    return t;
  };
  for (;;) {
    const unsigned long long kids = __ballot(n_par == cur && lane > last_child);
    const int c = kids ? __ffsll((long long)kids) - 1 : -1;  // the next child to test; -1: draw here
    const float qv = c < 0 ? 0.f : lane_value(n_q, c);
    const int tk = c < 0 ? -1 : lane_value(n_tok, c);
    if (c < 0) {
      if (have_total) break;
    } else {
      last_child = c;
      const double p0 = lane_value(n_p0, c), u = (double)lane_value(n_u0, c);
      double p, qd;  // qd: the probability this sibling was drawn with
      if constexpr (kWor) {
        p = node_weight_wor(p0, qv, tk, nres, Zs, ql);
        qd = in_list(tk, rej, cur_len) ? 0.0 : (double)qv * cur_fac;
      } else {
        p = node_weight(p0, qv, nres, Zs);
        qd = (double)qv;
      }
      if (u * qd < p) {
        cur = c;
        ++depth;
        nres = 0;
        have_total = false;
        cur_len = 0; cur_fac = 1.0; rej_mass = 0.0;
        if (writer && tid == 0) P.accept_mask[row0 + c] = 1;
        continue;
      }
      // the next residual level subtracts the distribution this sibling was drawn from
      if constexpr (kWor) {
        qlen[nres] = cur_len;
        qfac[nres] = cur_fac;
      }
    }

    // The total over the vocabulary of the current level's weights (draw), or of the next one's before it is normalised
    // (rejection): s_tot per slice and their sum in slice order.
    const int level = c < 0 ? nres : nres + 1;
    const bool raw = c >= 0;
    for (bool done = false; !done;) {
      const int s0 = solo ? 0 : slice, s1 = solo ? S : slice + 1;
      for (int sl = s0; sl < s1; ++sl) park_share(sl, level, raw);
      __syncthreads();
      done = true;
      if (solo) {
        if (tid < S) s_tot[tid] = slice_sum(tid);
        __syncthreads();
      } else {
        unsigned long long* ex = P.exch + (size_t)(2 * b + (sweeps & 1)) * 2 * S;
        if (wv == 0) {
          // lanes 0 .. S - 1 carry the lower halves of the slices' sums, lanes 16 .. 16 + S - 1 the upper ones
          const double own = slice_sum(slice);
          const unsigned long long bits = __builtin_bit_cast(unsigned long long, own);
          const unsigned tag = (unsigned)sweeps + 1;
          const int of = lane & (kTreeMaxSlices - 1), half = lane / kTreeMaxSlices;
          const bool word = half < 2 && of < S;
          if (word && of == slice)
            store_word(&ex[half * S + of], ((unsigned long long)tag << 32) | (half ? bits >> 32 : bits & 0xffffffffull));
          unsigned long long u = 0;
          const bool wanted = word && of != slice;
          for (int polls = 0;;) {
            if (wanted && (unsigned)(u >> 32) != tag) u = load_word(&ex[half * S + of]);
            if (!__any(wanted && (unsigned)(u >> 32) != tag)) break;
            if (++polls > P.spin_limit) { s_fail = 1; break; }
            __builtin_amdgcn_s_sleep(1);
          }
          const unsigned part = of != slice ? (unsigned)u : half ? (unsigned)(bits >> 32) : (unsigned)bits;
          if (word) __builtin_memcpy((char*)s_tot + 8 * of + 4 * half, &part, 4);
        }
        __syncthreads();
        if (s_fail) {
          // A workgroup of the request has not arrived within the bound (the GPU is shared and they are not all resident,
          // or one of them gave up earlier): this one, which holds the whole walk state like every workgroup, repeats the
          // sweep over the entire vocabulary and finishes the request by itself - same sums in the same order, so the same
          // result.  Others that wait for it run into their own bound and do likewise; what several then write is the same.
          solo = true;
          done = false;
          __syncthreads();  // s_share and s_tot are about to be rewritten
        }
      }
    }
    ++sweeps;
    total = 0.0;
    for (int sl = 0; sl < S; ++sl) total += s_tot[sl];
    if (c < 0) break;

    have_total = total > 0.0;  // otherwise the residual vanished: the distribution is left as it was
    if (have_total) {
      Zs[nres] = total;
      invZs[nres] = 1.0 / total;
      ++nres;
    }
    if constexpr (kWor) {
      if (!in_list(tk, rej, cur_len)) {
        // the rejected token leaves the distribution the later siblings were drawn from
        rej[cur_len] = tk;
        ++cur_len;
        rej_mass += (double)qv;
        const double left = 1.0 - rej_mass;
        cur_fac = left > 0.0 ? 1.0 / left : 0.0;
      }
    }
  }

  // ---- 3. inverse-CDF draw ------------------------------------------------------------------------
  const bool skip_last = have_total;  // the total at hand is that of the unnormalised last level
  const double thr = (double)lane_value(node ? s_u1[lane] : 0.f, cur) * total;
  int sl = -1;        // the slice that holds the crossing; if rounding left none, the last one with any weight
  double base = 0.0;  // the weights before it
  {
    double run = 0.0;
    for (int i = 0; i < S; ++i) {
      const double t = s_tot[i];
      if (t > 0.0) { sl = i; base = run; }
      run += t;
      if (t > 0.0 && run > thr) break;
    }
  }
  if (writer && tid == 0) P.accept_len[b] = depth;
  if (sl < 0) {  // no weight anywhere
    if (writer && tid == 0) P.next_token[b] = -1;
    return;
  }
  if (!solo && sl != slice) return;  // no barrier between workgroups follows
  if (tid == 0) { s_pick = 0x7fffffff; s_lastpos = -1; }
  __syncthreads();
  const int lo = slice_lo(sl), n_loc = slice_lo(sl + 1) - lo;
  int lastpos = -1;
  for_groups(sl, nres, skip_last, [&](int gi, const double* x) AURORA_INLINE {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (x[e] > 0.0) lastpos = max(lastpos, gi * kGroup + lane * 4 + e);
    const double sg = wave_sum((x[0] + x[1]) + (x[2] + x[3]));
    if (lane == 0) s_gsum[gi - lo] = sg;
  });
  lastpos = wave_max(lastpos);
  if (lane == 0) atomicMax(&s_lastpos, lastpos);
  __syncthreads();
  // scan of the slice's group sums: thread t owns groups 4t .. 4t+3
  double mine[4], loc = 0.0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int g = tid * 4 + i;
    mine[i] = g < n_loc ? s_gsum[g] : 0.0;
    loc += mine[i];
  }
  const double incl = wave_incl_scan(loc, lane);
  if (lane == kWave - 1) s_wtot[wv] = incl;
  __syncthreads();
  double excl = base + (incl - loc);
  for (int i = 0; i < kAccWaves; ++i)
    if (i < wv) excl += s_wtot[i];
  int found = 0x7fffffff;
  double before = 0.0;
  {
    double run = excl;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int g = tid * 4 + i;
      const double nxt = run + mine[i];
      if (g < n_loc && found == 0x7fffffff && mine[i] > 0.0 && nxt > thr) { found = g; before = run; }
      run = nxt;
    }
    if (found != 0x7fffffff) atomicMin(&s_pick, found);
  }
  __syncthreads();
  const int pick = s_pick;
  if (pick == found && found != 0x7fffffff) s_pick_prefix = before;
  __syncthreads();
  if (wv != 0) return;
  int token = s_lastpos;  // rounding left no crossing: the slice's largest token with positive weight
  if (pick != 0x7fffffff) {
    const float* lrow = P.logits + (row0 + cur) * V;
    const int v0 = (lo + pick) * kGroup + lane * 4;
    double x[4];
    weights(lane_load(lrow, q_row(P, row0 + cur), v0, V, vec_ok), v0, nres, skip_last, x);
    const double lane_tot = (x[0] + x[1]) + (x[2] + x[3]);
    const double lane_incl = wave_incl_scan(lane_tot, lane) + s_pick_prefix;
    const unsigned long long hit = __ballot(lane_incl > thr);
    const unsigned long long pos = __ballot(lane_tot > 0.0);
    if (hit) {
      const int hl = __ffsll((long long)hit) - 1;  // first lane whose running sum crosses
      const double r0 = __shfl(lane_incl - lane_tot, hl, kWave);
      const double y0 = __shfl(x[0], hl, kWave), y1 = __shfl(x[1], hl, kWave), y2 = __shfl(x[2], hl, kWave);
      int e_hit = 3;
      if (r0 + y0 > thr) e_hit = 0;
      else if (r0 + y0 + y1 > thr) e_hit = 1;
      else if (r0 + y0 + y1 + y2 > thr) e_hit = 2;
      const int cand = (lo + pick) * kGroup + hl * 4 + e_hit;
      if (cand < V) token = cand;
    } else if (pos) {
      const int pl = 63 - __clzll((long long)pos);
      int e_last = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (__shfl(x[e], pl, kWave) > 0.0) e_last = e;
      token = (lo + pick) * kGroup + pl * 4 + e_last;
    }
  }
  if (lane == 0) P.next_token[b] = token;
}

void accept_chain_geometry(int batch, int vocab, int* slices, int* gmul, int* ngroups) {
  const int ng = (vocab + kGroup - 1) / kGroup;
  // enough slices that a wavefront sweeps its share in one batch of four groups, within about two
  // workgroups per compute unit over the whole batch
  int s = (ng + 31) / 32;
  const int cap = (512 + batch - 1) / (batch > 0 ? batch : 1);
  if (s > cap) s = cap;
  if (s < 1) s = 1;
  if (s > 64) s = 64;
  *slices = s;
  *gmul = kGroup / kWave;
  *ngroups = ng;
}

// polls before a workgroup of a split tree walk stops waiting for the others (host-side setting, see the header)
static int g_tree_spin_limit = kSpinLimit;
void set_tree_spin_limit(int polls) { g_tree_spin_limit = polls < 0 ? kSpinLimit : polls; }

__global__ void zero_words_kernel(unsigned long long* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0ull;
}

int accept_tree_max_slices() { return kTreeMaxSlices; }

// Workgroups per request for a sampling tree walk: as many as leave every workgroup at least 16 groups
// to sweep, at most kTreeMaxSlices, and S * B within the number of compute units (all of them resident
// at once); 1 when that leaves fewer than two.  (Their words, 4 S per request, fit into the 2 ngroups doubles.)
// One workgroup that holds the whole vocabulary in registers is ahead of two that exchange their sums: 16 trees of 16 nodes over
// 12 000 ids 25.8 against 28.0 us, of 64 nodes 35.9 against 37.0 - but not without replacement, where a group takes longer: 16
// trees of 64 nodes over 8000 ids 53.0 against 49.7.
static int tree_slices_for(int B, int ngroups, bool wor, int cus) {
  if (!wor && ngroups <= held_groups(wor) * kAccWaves) return 1;
  int s = ngroups / 16;
  if (s > kTreeMaxSlices) s = kTreeMaxSlices;
  if (B > 0 && s > cus / B) s = cus / B;
  return s >= 2 ? s : 1;
}

// A request's only workgroup can form its rows' statistics from the logits (16 floats a lane and tile) and save a launch, while
// the tiles are few: each is a chain of reductions.  2 requests x 5 rows, step, us, with the launch and without: 2003 logits
// 44.8, 42.7, 4096 45.9, 47.1; 4 x 5 rows, 1024 26.9, 18.0 (with the shared launch in front, generic LM head), 8192 65.8, 73.7.
// A wavefront forms the tiles of every eighth row one after the other, where the launch has all of them side by side - until
// there are enough of them to fill the chip either way, and the launch only reads the logits once more.  LM head and acceptance, us, with the
// launch and without, by tiles a wavefront: two (16 rows x 1024) 1 request 17.8, 15.8, three (24 x 1024) 1 request 19.5, 19.3,
// 32 requests 27.8, 26.7; four (32 x 1024) 1 request 21.6, 22.7, (16 x 2048) 8 requests 19.1, 21.2, 64 requests 31.4, 30.8; eight
// (32 x 2048) 64 requests 45.9, 49.0, 128 requests 63.4, 58.4; sixteen (64 x 2048) 1 request 29.5, 53.2, 128 requests 105, 100.
bool accept_forms_stats(const AcceptLaunch& a) {
  const int chain = a.plan.n_tiles * ((a.Nq + kSweepThreads / kWave - 1) / (kSweepThreads / kWave));
  return (a.temperature > 0.f || a.temps) && !a.parents && a.plan.slices == 1 && a.plan.stat_tile == kRowStatTile &&
         a.plan.n_tiles <= kRowStatTiles && (chain <= 3 || a.B >= 128);
}

hipError_t launch_accept(const AcceptLaunch& a, hipStream_t st) {
  AcceptParams P = {};
  P.Nq = a.Nq; P.V = a.V; P.n_tiles = a.plan.n_tiles; P.temperature = a.temperature;
  P.logits = a.logits; P.pmax = a.pmax; P.psum = a.psum; P.parg = a.parg;
  P.tok = a.draft_tokens; P.q = a.draft_probs; P.un = a.uniforms; P.parents = a.parents;
  P.t2d = a.target_to_draft; P.Vq = a.target_to_draft ? a.Vd : a.V;
  P.accept_len = a.accept_len; P.next_token = a.next_token; P.accept_mask = a.accept_mask;
  P.p_at_draft = a.p_at_draft; P.row_lse = a.row_lse;
  P.slices = a.plan.slices; P.gmul = a.plan.gmul; P.ngroups = a.plan.ngroups;
  P.st_lse = a.st_lse; P.st_row = a.st_row; P.st_rej = a.st_rej; P.gsum = a.gsum; P.lastpos = a.lastpos;
  P.exch = (unsigned long long*)a.gsum;
  P.temps = a.temps;
  P.wor = a.wor;
  P.spin_limit = g_tree_spin_limit;
  const bool sampling = a.temperature > 0.f || a.temps != nullptr;  // per-request temperatures: the sampling kernels
  const bool chain_sampling = sampling && a.parents == nullptr;
  if (!chain_sampling) {
    const int ngroups = (a.V + kGroup - 1) / kGroup;
    if (sampling && ngroups > kMaxGroups) return hipErrorInvalidValue;
    int S = 1;
    if (sampling) {
      int cus = 0;
      if (hipError_t e = device_cu_count(&cus); e != hipSuccess) return e;
      S = tree_slices_for(a.B, ngroups, a.wor != 0, cus);
    }
    if (S > 1) {
      const int words = a.B * 4 * S;
      hipLaunchKernelGGL(zero_words_kernel, dim3((words + 255) / 256), dim3(256), 0, st, P.exch, words);
      if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    const bool held = (ngroups + S - 1) / S <= held_groups(P.wor != 0) * kAccWaves;
    // One workgroup that does not hold the vocabulary still keeps a total per slice, so that the draw re-reads one slice and
    // not the whole row: 64 groups, one round of loads for its wavefronts.  150 trees of four nodes over 151 936 ids: 257 us with
    // one slice, 188 with ten (222 with every group's sum kept from the last sweep); 256 of eight over 32 000: 84 and 77.
    P.solo_slices = held ? 1 : std::min(kTreeMaxSlices, (ngroups + 4 * kAccWaves - 1) / (4 * kAccWaves));
#define AURORA_TREE(HELD, WOR) hipLaunchKernelGGL((accept_tree_kernel<HELD, WOR>), dim3(S, a.B), dim3(kAccThreads), 0, st, P)
    if (held) {
      if (P.wor) AURORA_TREE(true, true); else AURORA_TREE(true, false);
    } else {
      if (P.wor) AURORA_TREE(false, true); else AURORA_TREE(false, false);
    }
#undef AURORA_TREE
    return hipGetLastError();
  }
  if (a.form_stats) hipLaunchKernelGGL(accept_chain_sweep<true>, dim3(1, a.B), dim3(kSweepThreads), 0, st, P);
  else hipLaunchKernelGGL(accept_chain_sweep<false>, dim3(P.slices, a.B), dim3(kSweepThreads), 0, st, P);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || P.slices == 1) return e;
  hipLaunchKernelGGL(accept_chain_pick, dim3(a.B), dim3(kSmallThreads), 0, st, P);
  return hipGetLastError();
}

}  // namespace aurora
