// The float attention kernels and what they share with the float GEMM: the float matrix instruction and its accumulator layout.  A
// header, since the kernels of wide heads are compiled apart from the others (attn_f32_wide.hip).
#pragma once
#include "common.h"

namespace beagle {
namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;

__device__ __forceinline__ f32x16_t mfma(float a, float b, const f32x16_t& c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16_t zero16() {
  f32x16_t z;
#pragma unroll
  for (int e = 0; e < 16; ++e) z[e] = 0.f;
  return z;
}
// row (A operand) or column of the 32 x 32 output that accumulator register e of lane half hf belongs to
__device__ __forceinline__ int acc_row(int e, int hf) { return 8 * (e >> 2) + 4 * hf + (e & 3); }

// ---------------------------------------------------------------------------
// Attention.  A workgroup owns 32 queries (keys) of one head; its four waves take blocks of 32 keys (queries) in turn
// and their results are merged in LDS in wave order.  As in the bf16 kernels a lane owns one query (key): scores come
// out of the matrix instruction with it as the column, and the probabilities go back in as the second product's operand
// without leaving their registers.  NC: 32-channel blocks of the head width.
// ---------------------------------------------------------------------------
// operand fragment of a row: channels 8 i + 4 hf + e at f[4 i + e], zeros past d.  FULL: d = 32 NC, nothing is past it.  (A select on
// a loaded value makes the wave wait for the load where it stands, ahead of whatever it would have requested next.  Without FULL the
// kernels therefore request a block where they need it: a block ahead, it saved nothing, cost registers, and at widths of 100 - 124
// spilled 41.  Steps with and without, us: 128 rows at width 36 47.1, 46.2; at 100 72.6, 71.8; 2 x 300 at 100 183, 178.)
template <int NC, bool FULL>
__device__ __forceinline__ void row_frag(const float* row, int d, int hf, float (&f)[16 * NC]) {
#pragma unroll
  for (int i = 0; i < 4 * NC; ++i) {
    const int c = 8 * i + 4 * hf;
    if constexpr (FULL) {
      const float4 v = *(const float4*)(row + c);
      f[4 * i] = v.x; f[4 * i + 1] = v.y; f[4 * i + 2] = v.z; f[4 * i + 3] = v.w;
      continue;
    }
    const float4 v = *(const float4*)(row + min(c, d - 4));
    const bool in = c < d;
    f[4 * i] = in ? v.x : 0.f; f[4 * i + 1] = in ? v.y : 0.f; f[4 * i + 2] = in ? v.z : 0.f; f[4 * i + 3] = in ? v.w : 0.f;
  }
}
// rows r0 + acc_row(e, hf) (clamped to n - 1) of channel c, for the product over rows; c is clamped by the caller
__device__ __forceinline__ void col_frag(const float* base, int64_t stride, int r0, int n, int c, int hf, float (&f)[16]) {
#pragma unroll
  for (int e = 0; e < 16; ++e) f[e] = base[min(r0 + acc_row(e, hf), n - 1) * stride + c];
}
template <int NC>
__device__ __forceinline__ f32x16_t dot_frags(const float (&a)[16 * NC], const float (&b)[16 * NC]) {
  f32x16_t s = zero16();
#pragma unroll
  for (int i = 0; i < 16 * NC; ++i) s = mfma(a[i], b[i], s);
  return s;
}
__device__ __forceinline__ float pair_sum(float v) { return v + __shfl_xor(v, 32, 64); }
__device__ __forceinline__ float pair_max(float v) { return fmaxf(v, __shfl_xor(v, 32, 64)); }

// Infinities and NaN behind the mask.  The second products multiply the rows that a query (key) must not see by a zero weight,
// which leaves nothing behind unless such a row is not finite.  Over the tiles that hold hidden pairs the waves therefore sum
// v * 0 over the fragments (a step of 128 rows takes 48 us with and without); where that is a NaN at the end, the wave starts over
// on plain code that reads only what each query (key) sees: the functions *_plain below, for which a lane keeps the row and the
// channels of its accumulators.
template <int N>
__device__ __forceinline__ void note_nonfinite(float& nf, const float (&f)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) nf = fmaf(f[i], 0.f, nf);
}
__device__ __forceinline__ bool any_nonfinite(float nf) { return __builtin_amdgcn_ballot_w64(nf != 0.f) != 0; }
// x . y over a head's channels, a lane pair's halves together
__device__ __forceinline__ float row_dot(const float* x, const float* y, int d, int hf) {
  float t = 0.f;
  for (int c = 4 * hf; c < d; c += 8) {
    const float4 u = *(const float4*)(x + c), v = *(const float4*)(y + c);
    t = fmaf(u.x, v.x, t); t = fmaf(u.y, v.y, t); t = fmaf(u.z, v.z, t); t = fmaf(u.w, v.w, t);
  }
  return pair_sum(t);
}
// o = o * keep + w * row where `take`
template <int NC>
__device__ __forceinline__ void add_row(f32x16_t (&o)[NC], bool take, float keep, float w, const float* row, int d, int hf) {
#pragma unroll
  for (int i = 0; i < 4 * NC; ++i) {
    const float4 x4 = *(const float4*)(row + min(8 * i + 4 * hf, d - 4));
    const float x[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float v = o[i >> 2][4 * (i & 3) + u];
      o[i >> 2][4 * (i & 3) + u] = take ? fmaf(w, x[u], v * keep) : v;
    }
  }
}

// A wave's accumulators [channel 32 cb + acc_row][row ql] -> LDS[row][channel], rows padded by one float
template <int NC>
__device__ __forceinline__ void park(float* buf, const f32x16_t (&o)[NC], int ql, int hf) {
#pragma unroll
  for (int cb = 0; cb < NC; ++cb)
#pragma unroll
    for (int e = 0; e < 16; ++e) buf[ql * (32 * NC + 1) + 32 * cb + acc_row(e, hf)] = o[cb][e];
}

template <int NC>
__device__ __forceinline__ void fwd_plain(const AttnArgs& a, const float* q, const float* K, const float* V, int64_t kvs, int first,
                                          int wg_lim, int lim, const uint32_t* trow, int hf, f32x16_t (&o)[NC], float& m, float& l) {
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) o[cb] = zero16();
  m = -INFINITY; l = 0.f;
#pragma unroll 1
  for (int j0 = first; j0 < wg_lim; j0 += 128)
#pragma unroll 1
    for (int j = j0; j < min(j0 + 32, wg_lim); ++j) {
      bool vis = j < lim;
      if (trow && j >= a.n_true && vis) { const int t = j - a.n_true; vis = ((trow[t >> 5] >> (t & 31)) & 1u) != 0; }
      const float s = a.scale * row_dot(q, K + j * kvs, a.d, hf);
      const float mn = vis ? fmaxf(m, s) : m, mb = mn == -INFINITY ? 0.f : mn;
      const float keep = expf(m - mb), p = expf(s - mb);
      l = vis ? l * keep + p : l;
      add_row<NC>(o, vis, keep, p, V + j * kvs, a.d, hf);
      m = mn;
    }
}

template <int NC, bool FULL>
__global__ __launch_bounds__(256, 1) void attn_fwd_f32_kernel(AttnArgs a) {
  __shared__ float ob[4][32 * (32 * NC + 1)];
  __shared__ float ms[4][32], ls[4][32];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), hf = lane >> 5, ql = lane & 31;
  const int h = blockIdx.y, b = blockIdx.z, g = h / (a.H / a.G), d = a.d;
  const int q0 = ((int)gridDim.x - 1 - (int)blockIdx.x) * 32;          // the queries that see the most keys first
  const SeqView sv = seq_view(a, b);
  if (q0 >= sv.S) return;                               // packed batch: a shorter entry
  const int q = q0 + ql, qc = min(q, sv.S - 1);
  const float* K = (const float*)a.k + (sv.kv0 * a.G + g) * d;
  const float* V = (const float*)a.v + (sv.kv0 * a.G + g) * d;
  const int64_t kvs = (int64_t)a.G * d;
  const float* Q = (const float*)a.q + ((sv.q0 + qc) * a.H + h) * d;
  // FULL: everything the wave's first block needs is requested at once, ahead of the mask's divisions (one trip to memory, not two),
  // and a next block's operands as soon as this one's are used
  float qf[16 * NC], kf[16 * NC], vf[NC][16];
  row_frag<NC, FULL>(Q, d, hf, qf);
  auto keys = [&](int j0) BEAGLE_INLINE_LAMBDA { row_frag<NC, FULL>(K + min(j0 + ql, sv.L - 1) * kvs, d, hf, kf); };
  auto values = [&](int j0) BEAGLE_INLINE_LAMBDA {
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) col_frag(V, kvs, j0, sv.L, min(32 * cb + ql, d - 1), hf, vf[cb]);
  };
  if constexpr (FULL) {
    if (sv.L > 0) { keys(32 * wave); values(32 * wave); }
    __builtin_amdgcn_sched_barrier(0);
  }
  const MaskParams mk = sample_mask(a, b);
  const int lim = q < sv.S ? row_limit(q, mk) : 0;
  const int wg_lim = row_limit(min(q0 + 32, sv.S) - 1, mk);            // limits never decrease with the query
  const int all_lim = min(row_limit(q0, mk), a.tree ? a.n_true : sv.L);   // keys below are seen by every query
  // draft-tree decode: keys at or past n_true are visible only where the query's tree row has a bit
  const uint32_t* trow = a.tree ? a.tree + (int64_t)qc * a.tree_words : nullptr;

  f32x16_t o[NC];
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) o[cb] = zero16();
  float m = -INFINITY, l = 0.f, nf = 0.f;
  for (int j0 = 32 * wave; j0 < wg_lim; j0 += 128) {
    if constexpr (!FULL) { keys(j0); values(j0); }
    f32x16_t s = dot_frags<NC>(kf, qf);                 // [key acc_row(e, hf)][query ql]
    if (FULL && j0 + 128 < wg_lim) keys(j0 + 128);
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int j = j0 + acc_row(e, hf);
      bool vis = j < lim;
      if (trow && j >= a.n_true && vis) { const int t = j - a.n_true; vis = ((trow[t >> 5] >> (t & 31)) & 1u) != 0; }
      s[e] = vis ? a.scale * s[e] : -INFINITY;
      mx = fmaxf(mx, s[e]);
    }
    const float mn = fmaxf(m, pair_max(mx));
    const float mb = mn == -INFINITY ? 0.f : mn;        // nothing visible so far: every p is exp(-inf) = 0
    const float alpha = expf(m - mb);
    float rs = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) { s[e] = expf(s[e] - mb); rs += s[e]; }
    l = l * alpha + pair_sum(rs);
    m = mn;
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
#pragma unroll
      for (int e = 0; e < 16; ++e) o[cb][e] *= alpha;
#pragma unroll
      for (int e = 0; e < 16; ++e) o[cb] = mfma(vf[cb][e], s[e], o[cb]);
    }
    if (j0 + 32 > all_lim) {
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) note_nonfinite(nf, vf[cb]);
    }
    if (FULL && j0 + 128 < wg_lim) values(j0 + 128);
  }
  if (any_nonfinite(nf)) fwd_plain<NC>(a, Q, K, V, kvs, 32 * wave, wg_lim, lim, trow, hf, o, m, l);
  park<NC>(ob[wave], o, ql, hf);
  if (hf == 0) { ms[wave][ql] = m; ls[wave][ql] = l; }
  __syncthreads();
  // 8 threads per query, every eighth channel each
  const int r = tid >> 3, p = q0 + r;
  if (p >= sv.S) return;
  float mm = fmaxf(fmaxf(ms[0][r], ms[1][r]), fmaxf(ms[2][r], ms[3][r])), w[4], lt = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) { w[i] = ms[i][r] == -INFINITY ? 0.f : expf(ms[i][r] - mm); lt += ls[i][r] * w[i]; }
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
  float* O = (float*)a.o + ((sv.q0 + p) * a.H + h) * d;
  for (int c = tid & 7; c < d; c += 8) {
    const int i = r * (32 * NC + 1) + c;
    O[c] = (((ob[0][i] * w[0] + ob[1][i] * w[1]) + ob[2][i] * w[2]) + ob[3][i] * w[3]) * inv;
  }
  if ((tid & 7) == 0) a.lse[sv.lse0 + h * sv.lse_hs + p] = lt > 0.f ? mm + logf(lt) : -INFINITY;
}

template <int NC>
__device__ __forceinline__ void dq_plain(const AttnArgs& a, const float* q, const float* g, float lse, float delta, const float* K,
                                         const float* V, int64_t kvs, int first, int wg_lim, int lim, int hf, f32x16_t (&dq)[NC]) {
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) dq[cb] = zero16();
#pragma unroll 1
  for (int j0 = first; j0 < wg_lim; j0 += 128)
#pragma unroll 1
    for (int j = j0; j < min(j0 + 32, wg_lim); ++j) {
      const float p = expf(a.scale * row_dot(q, K + j * kvs, a.d, hf) - lse);
      add_row<NC>(dq, j < lim, 1.f, p * (row_dot(g, V + j * kvs, a.d, hf) - delta), K + j * kvs, a.d, hf);
    }
}
// the (head, query block) pairs first, first + 4, ... of one key/value head, whose heads' query rows start at Q, dO, O
template <int NC>
__device__ __forceinline__ void dkv_plain(const AttnArgs& a, const SeqView& sv, const float* k, const float* v, const float* Q,
                                          const float* dO, const float* O, const float* lse, int64_t qs, int first, int pairs, int per,
                                          int qb0, int fq, int hf, f32x16_t (&dk)[NC], f32x16_t (&dv)[NC]) {
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) { dk[cb] = zero16(); dv[cb] = zero16(); }
#pragma unroll 1
  for (int it = first; it < pairs; it += 4) {
    const int hh = it / per, p0 = (qb0 + it % per) * 32;
#pragma unroll 1
    for (int p = p0; p < min(p0 + 32, sv.S); ++p) {
      const int64_t r = (int64_t)hh * a.d + p * qs;
      const float delta = row_dot(dO + r, O + r, a.d, hf);
      const float w = expf(a.scale * row_dot(Q + r, k, a.d, hf) - lse[hh * sv.lse_hs + p]);
      const float ds = w * (row_dot(dO + r, v, a.d, hf) - delta);
      add_row<NC>(dv, p >= fq, 1.f, w, dO + r, a.d, hf);
      add_row<NC>(dk, p >= fq, 1.f, ds, Q + r, a.d, hf);
    }
  }
}

// Both halves of the backward in one launch (they are independent: each forms delta = rowsum(dO * O) for itself).
//   blocks [0, n_dq)  : dQ of 32 queries of one head, over the keys they see; also stores delta
//   the rest          : dK, dV of 32 keys of one key/value head, over the (head, query block) pairs that see them
template <int NC, bool FULL>
__global__ __launch_bounds__(256, 1) void attn_bwd_f32_kernel(AttnArgs a, int n_dq) {
  __shared__ float ob[4][32 * (32 * NC + 1)];
  __shared__ float st[4][2][32];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), hf = lane >> 5, ql = lane & 31;
  const int d = a.d, rep = a.H / a.G;
  const int64_t kvs = (int64_t)a.G * d, qs = (int64_t)a.H * d;
  // the merged sums of the four waves, rows r0 .. of a tensor whose rows are `stride` apart
  auto rows_out = [&](float* out, int64_t stride, int rows, float scale) BEAGLE_INLINE_LAMBDA {
    __syncthreads();
    const int r = tid >> 3;
    if (r < rows)
      for (int c = tid & 7; c < d; c += 8) {
        const int i = r * (32 * NC + 1) + c;
        out[r * stride + c] = (((ob[0][i] + ob[1][i]) + ob[2][i]) + ob[3][i]) * scale;
      }
    __syncthreads();
  };
  if ((int)blockIdx.x < n_dq) {
    const int nq = (a.S + 31) / 32;
    const int row = blockIdx.x / nq, q0 = (nq - 1 - (int)blockIdx.x % nq) * 32;
    const int h = row % a.H, b = row / a.H, g = h / rep;
    const SeqView sv = seq_view(a, b);
    if (q0 >= sv.S) return;
    const int q = q0 + ql, qc = min(q, sv.S - 1);
    const int64_t qrow = ((sv.q0 + qc) * a.H + h) * d, li = sv.lse0 + h * sv.lse_hs + qc;
    const float* K = (const float*)a.k + (sv.kv0 * a.G + g) * d;
    const float* V = (const float*)a.v + (sv.kv0 * a.G + g) * d;
    // (FULL: one trip to memory, as in the forward)
    float qf[16 * NC], gf[16 * NC], kf[16 * NC], vf[16 * NC], kc[NC][16];
    auto rows = [&](int j0) BEAGLE_INLINE_LAMBDA {
      const int64_t jr = min(j0 + ql, sv.L - 1) * kvs;
      row_frag<NC, FULL>(K + jr, d, hf, kf);
      row_frag<NC, FULL>(V + jr, d, hf, vf);
    };
    auto cols = [&](int j0) BEAGLE_INLINE_LAMBDA {
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) col_frag(K, kvs, j0, sv.L, min(32 * cb + ql, d - 1), hf, kc[cb]);
    };
    float part = 0.f;
    const float lse = a.lse[li];
    {
      float of[16 * NC];
      row_frag<NC, FULL>((const float*)a.dout + qrow, d, hf, gf);
      row_frag<NC, FULL>((const float*)a.o + qrow, d, hf, of);
      row_frag<NC, FULL>((const float*)a.q + qrow, d, hf, qf);
      if constexpr (FULL) {
        if (sv.L > 0) { rows(32 * wave); cols(32 * wave); }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 0; i < 16 * NC; ++i) part = fmaf(gf[i], of[i], part);
    }
    const float delta = pair_sum(part);
    if (wave == 0 && hf == 0 && q < sv.S) a.delta[li] = delta;
    const MaskParams mk = sample_mask(a, b);
    const int lim = q < sv.S ? row_limit(q, mk) : 0;
    const int wg_lim = row_limit(min(q0 + 32, sv.S) - 1, mk), all_lim = row_limit(q0, mk);
    f32x16_t dq[NC];
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) dq[cb] = zero16();
    float nf = 0.f;
    for (int j0 = 32 * wave; j0 < wg_lim; j0 += 128) {
      if constexpr (!FULL) { rows(j0); cols(j0); }
      f32x16_t s = dot_frags<NC>(kf, qf);
      const f32x16_t dp = dot_frags<NC>(vf, gf);
      if (FULL && j0 + 128 < wg_lim) rows(j0 + 128);
#pragma unroll
      for (int e = 0; e < 16; ++e)
        s[e] = j0 + acc_row(e, hf) < lim ? expf(a.scale * s[e] - lse) * (dp[e] - delta) : 0.f;
#pragma unroll
      for (int cb = 0; cb < NC; ++cb)
#pragma unroll
        for (int e = 0; e < 16; ++e) dq[cb] = mfma(kc[cb][e], s[e], dq[cb]);
      if (j0 + 32 > all_lim) {
#pragma unroll
        for (int cb = 0; cb < NC; ++cb) note_nonfinite(nf, kc[cb]);
      }
      if (FULL && j0 + 128 < wg_lim) cols(j0 + 128);
    }
    if (any_nonfinite(nf))
      dq_plain<NC>(a, (const float*)a.q + qrow, (const float*)a.dout + qrow, lse, delta, K, V, kvs, 32 * wave, wg_lim, lim, hf, dq);
    park<NC>(ob[wave], dq, ql, hf);
    rows_out((float*)a.dq + ((sv.q0 + q0) * a.H + h) * d, qs, min(32, sv.S - q0), a.scale);
  } else {
    const int nk = (a.L + 31) / 32, n = (int)blockIdx.x - n_dq;
    const int row = n / nk, j0 = (n % nk) * 32, g = row % a.G, b = row / a.G;
    const SeqView sv = seq_view(a, b);
    if (j0 >= sv.L) return;
    const int j = j0 + ql;
    const int64_t kvrow = ((sv.kv0 + min(j, sv.L - 1)) * a.G + g) * d;
    float kf[16 * NC], vf[16 * NC];
    row_frag<NC, FULL>((const float*)a.k + kvrow, d, hf, kf);
    row_frag<NC, FULL>((const float*)a.v + kvrow, d, hf, vf);
    constexpr bool EARLY = NC <= 2;                  // the second products' operands are requested with the first ones'
    constexpr bool STATS_FIRST = !FULL && EARLY;     // delta is formed ahead of them: the selects have waited for its rows anyway
    if constexpr (!STATS_FIRST) __builtin_amdgcn_sched_barrier(0);
    const MaskParams mk = sample_mask(a, b);
    const int fq = j < sv.L ? first_query_seeing(j, mk) : sv.S;         // this lane's key is seen from here on
    const int all_q = first_query_seeing(min(j0 + 32, sv.L) - 1, mk);   // the workgroup's keys are all seen from here on
    const int qb0 = first_query_seeing(j0, mk) / 32, nqb = (sv.S + 31) / 32, per = nqb > qb0 ? nqb - qb0 : 0;
    f32x16_t dk[NC], dv[NC];
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) { dk[cb] = zero16(); dv[cb] = zero16(); }
    float nf = 0.f;
    for (int it = wave; it < per * rep; it += 4) {
      const int hh = it / per, p0 = (qb0 + it % per) * 32, h = g * rep + hh;
      const float* Q = (const float*)a.q + (sv.q0 * a.H + h) * d;
      const float* dO = (const float*)a.dout + (sv.q0 * a.H + h) * d;
      const int pc = min(p0 + ql, sv.S - 1);
      float qf[16 * NC], gf[16 * NC];
      row_frag<NC, FULL>(Q + pc * qs, d, hf, qf);
      row_frag<NC, FULL>(dO + pc * qs, d, hf, gf);
      const float lse = a.lse[sv.lse0 + h * sv.lse_hs + pc];
      float of[16 * NC], part = 0.f;
      row_frag<NC, FULL>((const float*)a.o + (sv.q0 * a.H + h) * d + pc * qs, d, hf, of);
      // delta, and both statistics to where the wave's other lanes find them (written and read by this wave only)
      auto stats = [&]() BEAGLE_INLINE_LAMBDA {
#pragma unroll
        for (int i = 0; i < 16 * NC; ++i) part = fmaf(gf[i], of[i], part);
        part = pair_sum(part);
        if (hf == 0) { st[wave][0][ql] = lse; st[wave][1][ql] = part; }
        __builtin_amdgcn_wave_barrier();
      };
      if constexpr (STATS_FIRST) stats();
      // the second products' operands: requested here where registers allow (head width up to 64)
      float cg[EARLY ? NC : 1][16], cq[EARLY ? NC : 1][16];
      if constexpr (EARLY) {
#pragma unroll
        for (int cb = 0; cb < NC; ++cb) {
          col_frag(dO, qs, p0, sv.S, min(32 * cb + ql, d - 1), hf, cg[cb]);
          col_frag(Q, qs, p0, sv.S, min(32 * cb + ql, d - 1), hf, cq[cb]);
        }
        if constexpr (!STATS_FIRST) __builtin_amdgcn_sched_barrier(0);
      }
      f32x16_t s = dot_frags<NC>(qf, kf);               // [query acc_row(e, hf)][key ql]
      f32x16_t dp = dot_frags<NC>(gf, vf);
      if constexpr (!STATS_FIRST) stats();
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int r = acc_row(e, hf), p = p0 + r;
        const bool vis = p >= fq && p < sv.S;           // a blind query (LSE -inf) is below fq of every key
        s[e] = vis ? expf(a.scale * s[e] - st[wave][0][r]) : 0.f;
        dp[e] = vis ? s[e] * (dp[e] - st[wave][1][r]) : 0.f;
      }
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) {
        constexpr int CB = EARLY ? 1 : 0;
        if constexpr (!EARLY) {
          col_frag(dO, qs, p0, sv.S, min(32 * cb + ql, d - 1), hf, cg[0]);
          col_frag(Q, qs, p0, sv.S, min(32 * cb + ql, d - 1), hf, cq[0]);
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) { dv[cb] = mfma(cg[CB * cb][e], s[e], dv[cb]); dk[cb] = mfma(cq[CB * cb][e], dp[e], dk[cb]); }
        if (p0 < all_q || p0 + 32 > sv.S) { note_nonfinite(nf, cg[CB * cb]); note_nonfinite(nf, cq[CB * cb]); }
      }
    }
    if (any_nonfinite(nf)) {
      const int64_t qh = (sv.q0 * a.H + g * rep) * d;                   // query 0 of the group's first head
      dkv_plain<NC>(a, sv, (const float*)a.k + kvrow, (const float*)a.v + kvrow, (const float*)a.q + qh, (const float*)a.dout + qh,
                    (const float*)a.o + qh, a.lse + sv.lse0 + g * rep * sv.lse_hs, qs, wave, per * rep, per, qb0, fq, hf, dk, dv);
    }
    const int64_t out0 = ((sv.kv0 + j0) * a.G + g) * d;
    park<NC>(ob[wave], dk, ql, hf);
    rows_out((float*)a.dk + out0, kvs, min(32, sv.L - j0), a.scale);
    park<NC>(ob[wave], dv, ql, hf);
    rows_out((float*)a.dv + out0, kvs, min(32, sv.L - j0), 1.f);
  }
}

// NC0 .. NC0 + 1 blocks of 32 channels
template <int NC0>
void launch_fwd(const AttnArgs& a, hipStream_t s) {
  const dim3 grid((a.S + 31) / 32, a.H, a.B), wg(256);
  auto go = [&](auto nc_) {
    constexpr int NC = decltype(nc_)::value;
    if (a.d == 32 * NC) hipLaunchKernelGGL((attn_fwd_f32_kernel<NC, true>), grid, wg, 0, s, a);
    else hipLaunchKernelGGL((attn_fwd_f32_kernel<NC, false>), grid, wg, 0, s, a);
  };
  if (a.d <= 32 * NC0) go(int_c<NC0>{}); else go(int_c<NC0 + 1>{});
}
template <int NC0>
void launch_bwd(const AttnArgs& a, hipStream_t s) {
  const int n_dq = ((a.S + 31) / 32) * a.H * a.B, n_dkv = ((a.L + 31) / 32) * a.G * a.B;
  const dim3 grid(n_dq + n_dkv), wg(256);
  auto go = [&](auto nc_) {
    constexpr int NC = decltype(nc_)::value;
    if (a.d == 32 * NC) hipLaunchKernelGGL((attn_bwd_f32_kernel<NC, true>), grid, wg, 0, s, a, n_dq);
    else hipLaunchKernelGGL((attn_bwd_f32_kernel<NC, false>), grid, wg, 0, s, a, n_dq);
  };
  if (a.d <= 32 * NC0) go(int_c<NC0>{}); else go(int_c<NC0 + 1>{});
}

}  // namespace
// heads of 68 .. 128 channels
void launch_attn_fwd_f32_wide(const AttnArgs& a, hipStream_t s);
void launch_attn_bwd_f32_wide(const AttnArgs& a, hipStream_t s);
}  // namespace beagle
