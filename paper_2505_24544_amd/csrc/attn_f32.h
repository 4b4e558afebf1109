// The float attention kernels, and the float matrix instruction that the float GEMM (f32_kernels.hip) shares with them.
#pragma once
#include "common.h"
#include "f32_plan.h"

namespace beagle {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

// v_mfma_f32_16x16x4_f32: lane (n, g) = (lane % 16, lane / 16) supplies row (column) n at k = g; accumulator e is row 4 g + e, column n
__device__ __forceinline__ f32x4_t mfma16(float a, float b, const f32x4_t& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4_t zero4() { return f32x4_t{0.f, 0.f, 0.f, 0.f}; }

// ---------------------------------------------------------------------------
// Attention.  A workgroup owns 16 queries (keys) of one head; its eight waves take blocks of 16 keys (queries) in turn
// and their results are merged in LDS in wave order.  As in the bf16 kernels a lane owns one query (key): scores come
// out of the matrix instruction with it as the column, and the probabilities go back in as the second product's operand
// without leaving their registers.  NC: 32-channel blocks of the head width.
//
// What bounds these kernels is one wave's serial chain, behind one trip to memory: the problems are small (128 rows of 4 heads are
// 32 workgroups).  Blocks of 16 x 16 and eight waves make the chain a quarter of what blocks of 32 x 32 and four waves had (at 64
// channels 32 and 64 instructions of 32 cycles, forward and dK/dV, for 64 and 128 of 64), and reading four channels of a row at once
// (below) takes 28 requests instead of 104.  Steps, us, before and now: 128 rows at 4 x 64 channels 46.6, 39.4, at 4 x 128 75.5, 62.4;
// 2 x 300 at 4 x 64 in 2 groups 95.7, 62.7; 24 at 4 x 32 30.3, 28.9 (the GEMMs the same on both sides).
// ---------------------------------------------------------------------------
constexpr int AW = 8;                                   // waves of a workgroup
constexpr int AT = 16;                                  // queries (keys) of a workgroup, keys (queries) of a wave's block

// operand fragment of a row: channels 16 j + 4 g + e at f[4 j + e], zeros past d.  FULL: d = 32 NC, nothing is past it.  (A select on
// a loaded value makes the wave wait for the load where it stands, ahead of whatever it would have requested next.  Without FULL the
// kernels therefore request a block where they need it.)
template <int NC, bool FULL>
__device__ __forceinline__ void row_frag(const float* row, int d, int g, float (&f)[8 * NC]) {
#pragma unroll
  for (int j = 0; j < 2 * NC; ++j) {
    const int c = 16 * j + 4 * g;
    if constexpr (FULL) {
      const float4 v = *(const float4*)(row + c);
      f[4 * j] = v.x; f[4 * j + 1] = v.y; f[4 * j + 2] = v.z; f[4 * j + 3] = v.w;
      continue;
    }
    const float4 v = *(const float4*)(row + min(c, d - 4));
    const bool in = c < d;
    f[4 * j] = in ? v.x : 0.f; f[4 * j + 1] = in ? v.y : 0.f; f[4 * j + 2] = in ? v.z : 0.f; f[4 * j + 3] = in ? v.w : 0.f;
  }
}
// Operand of the product over rows: rows r0 + 4 g + e (clamped to n - 1) at f[cb][e].  Which channel a lane's n stands for in
// instruction cb is free: in a block of 64 channels it is 4 n + cb, so that one 16-byte load feeds four instructions, in a last block
// of 32 it is 2 n + cb.  Accumulator e of instruction cb is then channel 16 g + 4 e + cb (8 g + 2 e + cb) of its block.  Channels past
// d repeat others; they are never stored.
template <int NC>
__device__ __forceinline__ void col_frag(const float* base, int64_t stride, int r0, int n, int nl, int g, int d, float (&f)[2 * NC][4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float* row = base + min(r0 + 4 * g + e, n - 1) * stride;
#pragma unroll
    for (int b = 0; b < NC / 2; ++b) {
      const float4 v = *(const float4*)(row + min(64 * b + 4 * nl, d - 4));
      f[4 * b][e] = v.x; f[4 * b + 1][e] = v.y; f[4 * b + 2][e] = v.z; f[4 * b + 3][e] = v.w;
    }
    if constexpr (NC & 1) {
      const float2 v = *(const float2*)(row + min(32 * (NC - 1) + 2 * nl, d - 2));
      f[2 * NC - 2][e] = v.x; f[2 * NC - 1][e] = v.y;
    }
  }
}
template <int NC>
__device__ __forceinline__ f32x4_t dot_frags(const float (&a)[8 * NC], const float (&b)[8 * NC]) {
  f32x4_t s = zero4();
#pragma unroll
  for (int i = 0; i < 8 * NC; ++i) s = mfma16(a[i], b[i], s);
  return s;
}
// over the four lanes that hold a row (column) together
__device__ __forceinline__ float quad_sum(float v) { v += __shfl_xor(v, 16, 64); return v + __shfl_xor(v, 32, 64); }
__device__ __forceinline__ float quad_max(float v) { v = fmaxf(v, __shfl_xor(v, 16, 64)); return fmaxf(v, __shfl_xor(v, 32, 64)); }

// Infinities and NaN behind the mask.  The second products multiply the rows that a query (key) must not see by a zero weight,
// which leaves nothing behind unless such a row is not finite.  Over the tiles that hold hidden pairs the waves therefore sum
// v * 0 over the fragments (a step of 128 rows took 48 us with and without, in blocks of 32 x 32); where that is a NaN at the end, the wave starts over
// on plain code that reads only what each query (key) sees: the functions *_plain below, for which a lane keeps the row and the
// channels of its accumulators.
template <int N>
__device__ __forceinline__ void note_nonfinite(float& nf, const float (&f)[N][4]) {
#pragma unroll
  for (int i = 0; i < 4 * N; ++i) nf = fmaf(f[i >> 2][i & 3], 0.f, nf);
}
__device__ __forceinline__ bool any_nonfinite(float nf) { return __builtin_amdgcn_ballot_w64(nf != 0.f) != 0; }
// x . y over a head's channels, the four lanes' shares together
__device__ __forceinline__ float row_dot(const float* x, const float* y, int d, int g) {
  float t = 0.f;
  for (int c = 4 * g; c < d; c += 16) {
    const float4 u = *(const float4*)(x + c), v = *(const float4*)(y + c);
    t = fmaf(u.x, v.x, t); t = fmaf(u.y, v.y, t); t = fmaf(u.z, v.z, t); t = fmaf(u.w, v.w, t);
  }
  return quad_sum(t);
}
// The accumulators of lane group g in channel order, four consecutive channels at a time: f(first channel, o[cb][e] of the four)
template <int NC, class F>
__device__ __forceinline__ void by_channels(int g, F&& f) {
  static_for<0, 4 * (NC / 2)>([&](auto i_) {
    constexpr int b = decltype(i_)::value / 4, e = decltype(i_)::value % 4;
    f(64 * b + 16 * g + 4 * e, int_c<4 * b>{}, int_c<e>{}, int_c<4 * b + 1>{}, int_c<e>{}, int_c<4 * b + 2>{}, int_c<e>{}, int_c<4 * b + 3>{}, int_c<e>{});
  });
  if constexpr (NC & 1)
    static_for<0, 2>([&](auto i_) {
      constexpr int e = 2 * decltype(i_)::value, c0 = 2 * NC - 2;
      f(32 * (NC - 1) + 8 * g + 2 * e, int_c<c0>{}, int_c<e>{}, int_c<c0 + 1>{}, int_c<e>{}, int_c<c0>{}, int_c<e + 1>{}, int_c<c0 + 1>{}, int_c<e + 1>{});
    });
}
#define BY_CHANNELS_ARGS int c, auto c0, auto e0, auto c1, auto e1, auto c2, auto e2, auto c3, auto e3
#define AT_CHANNEL(o, i) o[decltype(c##i)::value][decltype(e##i)::value]
// o = o * keep + w * row where `take`
template <int NC>
__device__ __forceinline__ void add_row(f32x4_t (&o)[2 * NC], bool take, float keep, float w, const float* row, int d, int g) {
  by_channels<NC>(g, [&](BY_CHANNELS_ARGS) BEAGLE_INLINE_LAMBDA {
    const float4 x = *(const float4*)(row + min(c, d - 4));
    auto upd = [&](float v, float xv) BEAGLE_INLINE_LAMBDA { return take ? fmaf(w, xv, v * keep) : v; };
    AT_CHANNEL(o, 0) = upd(AT_CHANNEL(o, 0), x.x); AT_CHANNEL(o, 1) = upd(AT_CHANNEL(o, 1), x.y);
    AT_CHANNEL(o, 2) = upd(AT_CHANNEL(o, 2), x.z); AT_CHANNEL(o, 3) = upd(AT_CHANNEL(o, 3), x.w);
  });
}
// A wave's accumulators -> LDS[row][channel], rows padded by four floats
template <int NC>
__device__ __forceinline__ void park(float* buf, const f32x4_t (&o)[2 * NC], int nl, int g) {
  by_channels<NC>(g, [&](BY_CHANNELS_ARGS) BEAGLE_INLINE_LAMBDA {
    *(float4*)(buf + nl * (32 * NC + 4) + c) = make_float4(AT_CHANNEL(o, 0), AT_CHANNEL(o, 1), AT_CHANNEL(o, 2), AT_CHANNEL(o, 3));
  });
}
#undef AT_CHANNEL
#undef BY_CHANNELS_ARGS

template <int NC>
__device__ __forceinline__ void fwd_plain(const AttnArgs& a, const float* q, const float* K, const float* V, int64_t kvs, int first,
                                          int wg_lim, int lim, const uint32_t* trow, int g, f32x4_t (&o)[2 * NC], float& m, float& l) {
#pragma unroll
  for (int cb = 0; cb < 2 * NC; ++cb) o[cb] = zero4();
  m = -INFINITY; l = 0.f;
#pragma unroll 1
  for (int j0 = first; j0 < wg_lim; j0 += AW * AT)
#pragma unroll 1
    for (int j = j0; j < min(j0 + AT, wg_lim); ++j) {
      bool vis = j < lim;
      if (trow && j >= a.n_true && vis) { const int t = j - a.n_true; vis = ((trow[t >> 5] >> (t & 31)) & 1u) != 0; }
      const float s = a.scale * row_dot(q, K + j * kvs, a.d, g);
      const float mn = vis ? fmaxf(m, s) : m, mb = mn == -INFINITY ? 0.f : mn;
      const float keep = expf(m - mb), p = expf(s - mb);
      l = vis ? l * keep + p : l;
      add_row<NC>(o, vis, keep, p, V + j * kvs, a.d, g);
      m = mn;
    }
}

template <int NC, bool FULL>
__global__ __launch_bounds__(64 * AW, 1) void attn_fwd_f32_kernel(AttnArgs a, int last) {
  constexpr int LD = 32 * NC + 4;
  __shared__ __attribute__((aligned(16))) float ob[AW][AT * LD];
  __shared__ float ms[AW][AT], ls[AW][AT];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, nl = lane & 15;
  const int h = blockIdx.y, b = blockIdx.z, kvh = h / (a.H / a.G), d = a.d;
  const int q0 = (last - (int)blockIdx.x) * AT;                        // the queries that see the most keys first
  const SeqView sv = seq_view(a, b);
  if (q0 >= sv.S) return;                               // packed batch: a shorter entry
  const int q = q0 + nl, qc = min(q, sv.S - 1);
  const float* K = (const float*)a.k + (sv.kv0 * a.G + kvh) * d;
  const float* V = (const float*)a.v + (sv.kv0 * a.G + kvh) * d;
  const int64_t kvs = (int64_t)a.G * d;
  const float* Q = (const float*)a.q + ((sv.q0 + qc) * a.H + h) * d;
  // FULL: everything the wave's first block needs is requested at once, ahead of the mask's divisions (one trip to memory, not two),
  // and a next block's operands as soon as this one's are used
  float qf[8 * NC], kf[8 * NC], vf[2 * NC][4];
  row_frag<NC, FULL>(Q, d, g, qf);
  auto keys = [&](int j0) BEAGLE_INLINE_LAMBDA { row_frag<NC, FULL>(K + min(j0 + nl, sv.L - 1) * kvs, d, g, kf); };
  auto values = [&](int j0) BEAGLE_INLINE_LAMBDA { col_frag<NC>(V, kvs, j0, sv.L, nl, g, d, vf); };
  if constexpr (FULL) {
    if (sv.L > 0) { keys(AT * wave); values(AT * wave); }
    __builtin_amdgcn_sched_barrier(0);
  }
  const MaskParams mk = sample_mask(a, b);
  const int lim = q < sv.S ? row_limit(q, mk) : 0;
  const int wg_lim = row_limit(min(q0 + AT, sv.S) - 1, mk);            // limits never decrease with the query
  const int all_lim = min(row_limit(q0, mk), a.tree ? a.n_true : sv.L);   // keys below are seen by every query
  // draft-tree decode: keys at or past n_true are visible only where the query's tree row has a bit
  const uint32_t* trow = a.tree ? a.tree + (int64_t)qc * a.tree_words : nullptr;

  f32x4_t o[2 * NC];
#pragma unroll
  for (int cb = 0; cb < 2 * NC; ++cb) o[cb] = zero4();
  float m = -INFINITY, l = 0.f, nf = 0.f;
  for (int j0 = AT * wave; j0 < wg_lim; j0 += AW * AT) {
    if constexpr (!FULL) { keys(j0); values(j0); }
    f32x4_t s = dot_frags<NC>(kf, qf);                  // [key 4 g + e][query nl]
    if (FULL && j0 + AW * AT < wg_lim) keys(j0 + AW * AT);
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int j = j0 + 4 * g + e;
      bool vis = j < lim;
      if (trow && j >= a.n_true && vis) { const int t = j - a.n_true; vis = ((trow[t >> 5] >> (t & 31)) & 1u) != 0; }
      s[e] = vis ? a.scale * s[e] : -INFINITY;
      mx = fmaxf(mx, s[e]);
    }
    const float mn = fmaxf(m, quad_max(mx));
    const float mb = mn == -INFINITY ? 0.f : mn;        // nothing visible so far: every p is exp(-inf) = 0
    const float alpha = expf(m - mb);
    float rs = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) { s[e] = expf(s[e] - mb); rs += s[e]; }
    l = l * alpha + quad_sum(rs);
    m = mn;
#pragma unroll
    for (int cb = 0; cb < 2 * NC; ++cb) {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[cb][e] *= alpha;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int cb = 0; cb < 2 * NC; ++cb) o[cb] = mfma16(vf[cb][e], s[e], o[cb]);
    if (j0 + AT > all_lim) note_nonfinite(nf, vf);
    if (FULL && j0 + AW * AT < wg_lim) values(j0 + AW * AT);
  }
  if (any_nonfinite(nf)) fwd_plain<NC>(a, Q, K, V, kvs, AT * wave, wg_lim, lim, trow, g, o, m, l);
  park<NC>(ob[wave], o, nl, g);
  if (g == 0) { ms[wave][nl] = m; ls[wave][nl] = l; }
  __syncthreads();
  // 32 threads per query, four channels each
  const int r = tid >> 5, c = 4 * (tid & 31), p = q0 + r;
  if (p >= sv.S || c >= d) return;
  float mm = ms[0][r], lt = 0.f;
#pragma unroll
  for (int i = 1; i < AW; ++i) mm = fmaxf(mm, ms[i][r]);
  float4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < AW; ++i) {
    const float w = ms[i][r] == -INFINITY ? 0.f : expf(ms[i][r] - mm);
    const float4 v = *(const float4*)&ob[i][r * LD + c];
    t.x += v.x * w; t.y += v.y * w; t.z += v.z * w; t.w += v.w * w;
    lt += ls[i][r] * w;
  }
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
  *(float4*)((float*)a.o + ((sv.q0 + p) * a.H + h) * d + c) = make_float4(t.x * inv, t.y * inv, t.z * inv, t.w * inv);
  if (c == 0) a.lse[sv.lse0 + h * sv.lse_hs + p] = lt > 0.f ? mm + logf(lt) : -INFINITY;
}

template <int NC>
__device__ __forceinline__ void dq_plain(const AttnArgs& a, const float* q, const float* go, float lse, float delta, const float* K,
                                         const float* V, int64_t kvs, int first, int wg_lim, int lim, int g, f32x4_t (&dq)[2 * NC]) {
#pragma unroll
  for (int cb = 0; cb < 2 * NC; ++cb) dq[cb] = zero4();
#pragma unroll 1
  for (int j0 = first; j0 < wg_lim; j0 += AW * AT)
#pragma unroll 1
    for (int j = j0; j < min(j0 + AT, wg_lim); ++j) {
      const float p = expf(a.scale * row_dot(q, K + j * kvs, a.d, g) - lse);
      add_row<NC>(dq, j < lim, 1.f, p * (row_dot(go, V + j * kvs, a.d, g) - delta), K + j * kvs, a.d, g);
    }
}
// the (head, query block) pairs first, first + AW, ... of one key/value head, whose heads' query rows start at Q, dO, O
template <int NC>
__device__ __forceinline__ void dkv_plain(const AttnArgs& a, const SeqView& sv, const float* k, const float* v, const float* Q,
                                          const float* dO, const float* O, const float* lse, int64_t qs, int first, int pairs, int per,
                                          int qb0, int fq, int g, f32x4_t (&dk)[2 * NC], f32x4_t (&dv)[2 * NC]) {
#pragma unroll
  for (int cb = 0; cb < 2 * NC; ++cb) { dk[cb] = zero4(); dv[cb] = zero4(); }
#pragma unroll 1
  for (int it = first; it < pairs; it += AW) {
    const int hh = it / per, p0 = (qb0 + it % per) * AT;
#pragma unroll 1
    for (int p = p0; p < min(p0 + AT, sv.S); ++p) {
      const int64_t r = (int64_t)hh * a.d + p * qs;
      const float delta = row_dot(dO + r, O + r, a.d, g);
      const float w = expf(a.scale * row_dot(Q + r, k, a.d, g) - lse[hh * sv.lse_hs + p]);
      const float ds = w * (row_dot(dO + r, v, a.d, g) - delta);
      add_row<NC>(dv, p >= fq, 1.f, w, dO + r, a.d, g);
      add_row<NC>(dk, p >= fq, 1.f, ds, Q + r, a.d, g);
    }
  }
}

// Both halves of the backward in one launch (they are independent: each forms delta = rowsum(dO * O) for itself).
//   blocks [0, part.n_first) : dQ of 16 queries of one head, over the keys they see; also stores delta
//   the rest                 : dK, dV of 16 keys of one key/value head, over the (head, query block) pairs that see them
template <int NC, bool FULL>
__global__ __launch_bounds__(64 * AW, 1) void attn_bwd_f32_kernel(AttnArgs a, GridPart part) {
  constexpr int LD = 32 * NC + 4;
  __shared__ __attribute__((aligned(16))) float ob[AW][AT * LD];
  __shared__ __attribute__((aligned(16))) float st[AW][2][AT];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, nl = lane & 15;
  const int d = a.d, rep = a.H / a.G;
  const int64_t kvs = (int64_t)a.G * d, qs = (int64_t)a.H * d;
  // the merged sums of the waves, rows r0 .. of a tensor whose rows are `stride` apart
  auto rows_out = [&](float* out, int64_t stride, int rows, float scale) BEAGLE_INLINE_LAMBDA {
    __syncthreads();
    const int r = tid >> 5, c = 4 * (tid & 31);
    if (r < rows && c < d) {
      float4 t = *(const float4*)&ob[0][r * LD + c];
#pragma unroll
      for (int i = 1; i < AW; ++i) {
        const float4 v = *(const float4*)&ob[i][r * LD + c];
        t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
      }
      *(float4*)(out + r * stride + c) = make_float4(t.x * scale, t.y * scale, t.z * scale, t.w * scale);
    }
  };
  if (blockIdx.x < part.n_first) {
    const uint32_t nq = (a.S + AT - 1) / AT, at = part.blk0 + blockIdx.x, row = part.row0 + at / nq;
    const int q0 = (int)(nq - 1 - at % nq) * AT, h = row % (uint32_t)a.H, b = row / (uint32_t)a.H, kvh = h / rep;
    const SeqView sv = seq_view(a, b);
    if (q0 >= sv.S) return;
    const int q = q0 + nl, qc = min(q, sv.S - 1);
    const int64_t qrow = ((sv.q0 + qc) * a.H + h) * d, li = sv.lse0 + h * sv.lse_hs + qc;
    const float* K = (const float*)a.k + (sv.kv0 * a.G + kvh) * d;
    const float* V = (const float*)a.v + (sv.kv0 * a.G + kvh) * d;
    // (FULL: one trip to memory, as in the forward)
    float qf[8 * NC], gf[8 * NC], kf[8 * NC], vf[8 * NC], kc[2 * NC][4];
    auto rows = [&](int j0) BEAGLE_INLINE_LAMBDA {
      const int64_t jr = min(j0 + nl, sv.L - 1) * kvs;
      row_frag<NC, FULL>(K + jr, d, g, kf);
      row_frag<NC, FULL>(V + jr, d, g, vf);
    };
    auto cols = [&](int j0) BEAGLE_INLINE_LAMBDA { col_frag<NC>(K, kvs, j0, sv.L, nl, g, d, kc); };
    float part = 0.f;
    const float lse = a.lse[li];
    {
      float of[8 * NC];
      row_frag<NC, FULL>((const float*)a.dout + qrow, d, g, gf);
      row_frag<NC, FULL>((const float*)a.o + qrow, d, g, of);
      row_frag<NC, FULL>((const float*)a.q + qrow, d, g, qf);
      if constexpr (FULL) {
        if (sv.L > 0) { rows(AT * wave); cols(AT * wave); }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 0; i < 8 * NC; ++i) part = fmaf(gf[i], of[i], part);
    }
    const float delta = quad_sum(part);
    if (wave == 0 && g == 0 && q < sv.S) a.delta[li] = delta;
    const MaskParams mk = sample_mask(a, b);
    const int lim = q < sv.S ? row_limit(q, mk) : 0;
    const int wg_lim = row_limit(min(q0 + AT, sv.S) - 1, mk), all_lim = row_limit(q0, mk);
    f32x4_t dq[2 * NC];
#pragma unroll
    for (int cb = 0; cb < 2 * NC; ++cb) dq[cb] = zero4();
    float nf = 0.f;
    for (int j0 = AT * wave; j0 < wg_lim; j0 += AW * AT) {
      if constexpr (!FULL) { rows(j0); cols(j0); }
      f32x4_t s = dot_frags<NC>(kf, qf);
      const f32x4_t dp = dot_frags<NC>(vf, gf);
      if (FULL && j0 + AW * AT < wg_lim) rows(j0 + AW * AT);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        s[e] = j0 + 4 * g + e < lim ? expf(a.scale * s[e] - lse) * (dp[e] - delta) : 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int cb = 0; cb < 2 * NC; ++cb) dq[cb] = mfma16(kc[cb][e], s[e], dq[cb]);
      if (j0 + AT > all_lim) note_nonfinite(nf, kc);
      if (FULL && j0 + AW * AT < wg_lim) cols(j0 + AW * AT);
    }
    if (any_nonfinite(nf))
      dq_plain<NC>(a, (const float*)a.q + qrow, (const float*)a.dout + qrow, lse, delta, K, V, kvs, AT * wave, wg_lim, lim, g, dq);
    park<NC>(ob[wave], dq, nl, g);
    rows_out((float*)a.dq + ((sv.q0 + q0) * a.H + h) * d, qs, min(AT, sv.S - q0), a.scale);
  } else {
    const uint32_t nk = (a.L + AT - 1) / AT, at = part.blk1 + (blockIdx.x - part.n_first), row = part.row1 + at / nk;
    const int j0 = (int)(at % nk) * AT, kvh = row % (uint32_t)a.G, b = row / (uint32_t)a.G;
    const SeqView sv = seq_view(a, b);
    if (j0 >= sv.L) return;
    const int j = j0 + nl;
    const int64_t kvrow = ((sv.kv0 + min(j, sv.L - 1)) * a.G + kvh) * d;
    float kf[8 * NC], vf[8 * NC];
    row_frag<NC, FULL>((const float*)a.k + kvrow, d, g, kf);
    row_frag<NC, FULL>((const float*)a.v + kvrow, d, g, vf);
    if constexpr (FULL) __builtin_amdgcn_sched_barrier(0);
    const MaskParams mk = sample_mask(a, b);
    const int fq = j < sv.L ? first_query_seeing(j, mk) : sv.S;         // this lane's key is seen from here on
    const int all_q = first_query_seeing(min(j0 + AT, sv.L) - 1, mk);   // the workgroup's keys are all seen from here on
    const int qb0 = first_query_seeing(j0, mk) / AT, nqb = (sv.S + AT - 1) / AT, per = nqb > qb0 ? nqb - qb0 : 0;
    f32x4_t dk[2 * NC], dv[2 * NC];
#pragma unroll
    for (int cb = 0; cb < 2 * NC; ++cb) { dk[cb] = zero4(); dv[cb] = zero4(); }
    float nf = 0.f;
    for (int it = wave; it < per * rep; it += AW) {
      const int hh = it / per, p0 = (qb0 + it % per) * AT, h = kvh * rep + hh;
      const float* Q = (const float*)a.q + (sv.q0 * a.H + h) * d;
      const float* dO = (const float*)a.dout + (sv.q0 * a.H + h) * d;
      const int pc = min(p0 + nl, sv.S - 1);
      float qf[8 * NC], gf[8 * NC], of[8 * NC], cg[2 * NC][4], cq[2 * NC][4];
      row_frag<NC, FULL>(Q + pc * qs, d, g, qf);
      row_frag<NC, FULL>(dO + pc * qs, d, g, gf);
      const float lse = a.lse[sv.lse0 + h * sv.lse_hs + pc];
      row_frag<NC, FULL>((const float*)a.o + (sv.q0 * a.H + h) * d + pc * qs, d, g, of);
      auto cols = [&]() BEAGLE_INLINE_LAMBDA {
        col_frag<NC>(dO, qs, p0, sv.S, nl, g, d, cg);
        col_frag<NC>(Q, qs, p0, sv.S, nl, g, d, cq);
      };
      // the second products' operands: requested with the first ones' where registers allow (head width up to 64)
      constexpr bool EARLY = NC <= 2;
      if constexpr (EARLY) {
        cols();
        if constexpr (FULL) __builtin_amdgcn_sched_barrier(0);
      }
      f32x4_t s = dot_frags<NC>(qf, kf);                // [query 4 g + e][key nl]
      f32x4_t dp = dot_frags<NC>(gf, vf);
      // delta, and both statistics to where the wave's other lanes find them (written and read by this wave only)
      float part = 0.f;
#pragma unroll
      for (int i = 0; i < 8 * NC; ++i) part = fmaf(gf[i], of[i], part);
      part = quad_sum(part);
      if (g == 0) { st[wave][0][nl] = lse; st[wave][1][nl] = part; }
      __builtin_amdgcn_wave_barrier();
      if constexpr (!EARLY) cols();
      const float4 l4 = *(const float4*)&st[wave][0][4 * g], d4 = *(const float4*)&st[wave][1][4 * g];
      const float le[4] = {l4.x, l4.y, l4.z, l4.w}, de[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int p = p0 + 4 * g + e;
        const bool vis = p >= fq && p < sv.S;           // a blind query (LSE -inf) is below fq of every key
        s[e] = vis ? expf(a.scale * s[e] - le[e]) : 0.f;
        dp[e] = vis ? s[e] * (dp[e] - de[e]) : 0.f;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int cb = 0; cb < 2 * NC; ++cb) { dv[cb] = mfma16(cg[cb][e], s[e], dv[cb]); dk[cb] = mfma16(cq[cb][e], dp[e], dk[cb]); }
      if (p0 < all_q || p0 + AT > sv.S) { note_nonfinite(nf, cg); note_nonfinite(nf, cq); }
      __builtin_amdgcn_wave_barrier();                  // the statistics are read before the next block's are written
    }
    if (any_nonfinite(nf)) {
      const int64_t qh = (sv.q0 * a.H + kvh * rep) * d;                 // query 0 of the group's first head
      dkv_plain<NC>(a, sv, (const float*)a.k + kvrow, (const float*)a.v + kvrow, (const float*)a.q + qh, (const float*)a.dout + qh,
                    (const float*)a.o + qh, a.lse + sv.lse0 + kvh * rep * sv.lse_hs, qs, wave, per * rep, per, qb0, fq, g, dk, dv);
    }
    const int64_t out0 = ((sv.kv0 + j0) * a.G + kvh) * d;
    park<NC>(ob[wave], dk, nl, g);
    rows_out((float*)a.dk + out0, kvs, min(AT, sv.L - j0), a.scale);
    __syncthreads();
    park<NC>(ob[wave], dv, nl, g);
    rows_out((float*)a.dv + out0, kvs, min(AT, sv.L - j0), 1.f);
  }
}

}  // namespace
}  // namespace beagle
