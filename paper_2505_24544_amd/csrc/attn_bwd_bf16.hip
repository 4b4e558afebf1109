// Backward of the block-masked cross-attention for bf16, head width 128, on
// gfx950 MFMA, by recomputation from Q, K, V, O, dO and the stored LSE:
//   delta_p = sum_c dO_pc O_pc          P = exp(s - LSE)        dS = P * (dP - delta)
//   dQ = scale * dS K      dK = scale * dS^T Q      dV = P^T dO      dP = dO V^T
//
// No floating-point atomics (results are bitwise reproducible):
//
//  (1) dq kernel   one workgroup = 128 queries (64 in short batches, as in the
//      forward) of one (b, h), loop over the key tiles those queries can see.  A
//      lane owns ONE query, as in the forward: S^T = K Q^T and dP^T = V dO^T
//      come out with column q = lane % 32, so LSE and delta are per-lane scalars,
//      and dS^T goes straight from the accumulator registers into the B operand
//      of dQ^T += K^T dS^T.  The kernel also computes delta and stores it, with
//      -log2(e) * LSE, for kernel (2).
//
//  (2) dkv kernel  one workgroup = 128 keys of one (b, kv head), loop over the
//      H/G query heads of the group and over the query tiles that can see those
//      keys.  A lane owns ONE key: S = Q K^T and dP = dO V^T come out with
//      column j = lane % 32; P and dS go straight into the B operands of
//      dV^T += dO^T P and dK^T += Q^T dS.  LSE/delta of the tile's queries are
//      read from LDS (they index the accumulator registers here).  In short
//      grouped-query batches several workgroups share a key tile, and a third
//      kernel adds their sums in order.
//
// Tiles go from HBM/L2 straight into one of two LDS stages while the other is
// consumed; the swizzled tile layout (attn_tiles.h) serves both the whole-row
// fragments (k = channel) and the transpose fragments (k = row) without bank
// conflicts.
//
// Mask: query p sees key j iff j < row_limit(p) iff p >= first_query_seeing(j).
// Key tiles beyond a workgroup's last limit / query tiles before a key tile's
// first viewer are never visited (whole-tile skipping).
#include "attn_tiles.h"
#include "mfma_in_place.h"

namespace beagle {
using namespace tiles;

namespace bwd {
__device__ __forceinline__ float dot8(bf16x8_t a, bf16x8_t b) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) s = fmaf((float)a[i], (float)b[i], s);
  return s;
}
}  // namespace bwd

// ===========================================================================
// (1) dQ and delta
// ===========================================================================
namespace dqk {
constexpr int BJ = 64;
constexpr int TILE = BJ * HD;            // one K or V tile
}  // namespace dqk

// KH: key halves, as in the forward: with 2 a workgroup has 64 queries and two waves per 32 of them, one for either half of
// every tile; their dQ are added in LDS
template <int KH>
__global__ __launch_bounds__(256, 2) void attn_bwd_dq_bf16_kernel(AttnArgs a) {
  using namespace dqk;
  constexpr int BQ = 128 / KH, NJB = 2 / KH;      // queries per workgroup, 32-key blocks of a tile per wave
  args_at_hand(a);
  __shared__ __attribute__((aligned(1024))) bf16_t stage0[2 * TILE];
  __shared__ __attribute__((aligned(1024))) bf16_t stage1[2 * TILE];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), hf = lane >> 5, ql = lane & 31;
  const int nqt = (a.S + BQ - 1) / BQ;
  int row, tpos;
  map_block(blockIdx.x, a.H * a.B, row, tpos);
  const int qt = nqt - 1 - tpos;                  // heaviest (latest) query tiles first
  const int h = row % a.H, b = row / a.H, g = h / (a.H / a.G);
  const int qw = wave % (4 / KH), kw = wave / (4 / KH) * 32;   // this wave's queries, and its first key in a tile
  const int q0 = qt * BQ, qw0 = q0 + qw * 32, q = qw0 + ql;
  const SeqView sv = seq_view(a, b);
  if (q0 >= sv.S) return;                         // packed batch: this entry is shorter than the longest one
  const bool q_ok = q < sv.S;
  const int qc = q_ok ? q : sv.S - 1;
  const int64_t qrow = ((sv.q0 + qc) * a.H + h) * HD;
  const bf16_t* Qg = (const bf16_t*)a.q + qrow;
  const bf16_t* Og = (const bf16_t*)a.o + qrow;
  const bf16_t* dOg = (const bf16_t*)a.dout + qrow;
  const int64_t kvs = (int64_t)a.G * HD;
  const __amdgpu_buffer_rsrc_t krs = rows_rsrc((const bf16_t*)a.k + (sv.kv0 * a.G + g) * HD, sv.L, kvs);
  const __amdgpu_buffer_rsrc_t vrs = rows_rsrc((const bf16_t*)a.v + (sv.kv0 * a.G + g) * HD, sv.L, kvs);
  const int64_t li = sv.lse0 + h * sv.lse_hs + qc;

  auto fetch = [&](bf16_t* st, int jt) {
    load_rows<BJ>(st, krs, kvs, jt * BJ, tid);
    load_rows<BJ>(st + TILE, vrs, kvs, jt * BJ, tid);
  };
  // The first K/V tile, the LSE and this lane's own rows are requested one behind the other and before the mask's
  // arithmetic: one trip to memory for all of them (measured per workgroup: 9 300 cycles until the rows are there,
  // 3 300 more when the LSE is only asked for then), with the integer divisions of the mask running meanwhile.  Tile 0
  // exists unless no query of the workgroup sees any key; then its rows are fetched for nothing.
  fetch(stage0, 0);
  const float lse = a.lse[li];
  bf16x8_t qf[8], dof[8], of[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    qf[s] = *(const bf16x8_t*)(Qg + 16 * s + 8 * hf);
    dof[s] = *(const bf16x8_t*)(dOg + 16 * s + 8 * hf);
    of[s] = *(const bf16x8_t*)(Og + 16 * s + 8 * hf);
  }
  __builtin_amdgcn_sched_barrier(0);

  const MaskParams mk = sample_mask(a, b);
  const int lim = q_ok ? row_limit(q, mk) : 0;
  const int wg_lim = row_limit(min(q0 + BQ, sv.S) - 1, mk);
  const int wave_hi = qw0 < sv.S ? row_limit(min(qw0 + 32, sv.S) - 1, mk) : 0;
  const int wave_lo = qw0 < sv.S ? row_limit(qw0, mk) : 0;
  const int ntiles = (wg_lim + BJ - 1) / BJ;
  __builtin_amdgcn_sched_barrier(0);

  float part = 0.f;
#pragma unroll
  for (int s = 0; s < 8; ++s) part += bwd::dot8(dof[s], of[s]);
  const float delta = half_pair_sum(part);
  if (q_ok && hf == 0 && kw == 0) { a.delta[li] = delta; a.nlse2[li] = -LOG2E * lse; }   // blind rows: +inf, masked in the dK/dV kernel
  const float c2 = a.scale * LOG2E;
  const float lse2 = (lim > 0 ? lse : 0.f) * LOG2E;    // blind rows are fully masked below
  const FragOffs fo = make_frag_offs(lane);

  f32x16_t dq[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) dq[i][e] = 0.f;

  auto tile_step = [&](const bf16_t* cur, bf16_t* nxt, int jt) {
    const int j0 = jt * BJ + kw;
    if (j0 >= wave_hi) fetch(nxt, jt + 1);        // a wave that sees nothing of the tile only requests its share of the next
    if (j0 < wave_hi) {
      fetch(nxt, jt + 1);                         // issued between the MFMAs below
      const bf16_t* ks = cur + kw * HD;
      const bf16_t* vs = cur + TILE + kw * HD;
      f32x16_t st[NJB], dp[NJB];
#pragma unroll
      for (int jb = 0; jb < NJB; ++jb) {
#pragma unroll
        for (int e = 0; e < 16; ++e) { st[jb][e] = 0.f; dp[jb][e] = 0.f; }
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          st[jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(row_frag(ks, fo, jb, s), qf[s], st[jb], 0, 0, 0);
          dp[jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(row_frag(vs, fo, jb, s), dof[s], dp[jb], 0, 0, 0);
        }
      }
      pipeline_reads_mfma_loads<32 / KH, 1, 8>();
      __builtin_amdgcn_sched_barrier(0);
      // dS = P (dP - delta); key offsets inside the tile are compile-time constants, and only tiles that reach
      // past the smallest limit of the wave run the compares and selects (a scalar branch around them alone)
      float dsv[NJB][16];
#pragma unroll
      for (int jb = 0; jb < NJB; ++jb)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float p = __builtin_amdgcn_exp2f(st[jb][e] * c2 - lse2);
          dsv[jb][e] = p * (dp[jb][e] - delta);
        }
      if (j0 + 32 * NJB > wave_lo) {
        const int rel = lim - j0 - 4 * hf;
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (32 * jb + 8 * (e >> 2) + (e & 3) >= rel) dsv[jb][e] = 0.f;
      }
      uint32_t pk[NJB][8];
#pragma unroll
      for (int jb = 0; jb < NJB; ++jb)
#pragma unroll
        for (int e = 0; e < 16; e += 2) pk[jb][e >> 1] = cvt_pk(dsv[jb][e], dsv[jb][e + 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int jb = 0; jb < NJB; ++jb)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          union { uint32_t u[4]; bf16x8_t v; } sf;
#pragma unroll
          for (int i = 0; i < 4; ++i) sf.u[i] = pk[jb][4 * t + i];
#pragma unroll
          for (int cb = 0; cb < 4; ++cb)
            dq[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr_frag(ks, fo, 32 * jb + 16 * t, cb), sf.v, dq[cb], 0, 0, 0);
        }
      pipeline_reads_mfma<16 / KH, 2>();
      __builtin_amdgcn_sched_barrier(0);
    }
    wait_vmem();
    __syncthreads();
  };

  wait_vmem();
  __syncthreads();
  int jt = 0;
#pragma unroll 1
  for (; jt + 2 <= ntiles; jt += 2) {
    tile_step(stage0, stage1, jt);
    tile_step(stage1, stage0, jt + 1);
  }
  if (jt < ntiles) tile_step(stage0, stage1, jt);

  if constexpr (KH == 2) {
    float4* po = (float4*)stage0 + qw * 64 + lane;               // [16][2 waves][64 lanes]: 32 KB
    if (kw) {
#pragma unroll
      for (int i = 0; i < 16; ++i) po[128 * i] = float4{dq[i >> 2][4 * (i & 3)], dq[i >> 2][4 * (i & 3) + 1], dq[i >> 2][4 * (i & 3) + 2], dq[i >> 2][4 * (i & 3) + 3]};
    }
    __syncthreads();
    if (kw) return;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float4 v = po[128 * i];
      const float w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) dq[i >> 2][4 * (i & 3) + e] += w[e];
    }
  }

  // ---- dQ rows out, through LDS (the stages are free: the last step, or the prologue, ended with a barrier)
  {
    uint2 pq[16];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd)
        pq[4 * cb + qd] = make_uint2(cvt_pk(dq[cb][4 * qd] * a.scale, dq[cb][4 * qd + 1] * a.scale),
                                     cvt_pk(dq[cb][4 * qd + 2] * a.scale, dq[cb][4 * qd + 3] * a.scale));
    store_rows_via_lds((KH == 1 ? stage0 : stage1) + qw * 32 * HD, pq, lane, (bf16_t*)a.dq + ((sv.q0 + qw0) * a.H + h) * HD, (int64_t)a.H * HD,
                       sv.S - qw0);
  }
}

// ===========================================================================
// (2) dK and dV
// ===========================================================================
namespace dkv {
constexpr int BJ = 128, BQ = 64;
constexpr int TILE = BQ * HD;            // one Q or dO tile
constexpr int AHEAD = 4;                // MFMAs from an LDS fragment's read to its use
constexpr int SLOT = 2 * BJ * HD;        // floats of one partial result: dK, then dV of a key tile
// SPLIT: a key tile's (head, query tile) pairs are cut into chunks of `per_chunk`, up to `chunks` workgroups per tile
struct Split { float* part; int32_t chunks, per_chunk; };
// pairs of key tile j0, and the workgroups that share them (at least one: it writes the zeros of unseen keys)
__device__ __forceinline__ int tile_pairs(int j0, const MaskParams& mk, int S, int rep) {
  const int qt0 = first_query_seeing(j0, mk) / BQ, nqt = (S + BQ - 1) / BQ;
  return nqt > qt0 ? (nqt - qt0) * rep : 0;
}
__device__ __forceinline__ int tile_chunks(int pairs, int per_chunk) { return pairs > per_chunk ? (pairs + per_chunk - 1) / per_chunk : 1; }
}  // namespace dkv

template <bool SPLIT>
__global__ __launch_bounds__(256, 1) void attn_bwd_dkv_bf16_kernel(AttnArgs a, dkv::Split sp) {
  using namespace dkv;
  args_at_hand(a);
  __shared__ __attribute__((aligned(1024))) bf16_t stage0[2 * TILE];
  __shared__ __attribute__((aligned(1024))) bf16_t stage1[2 * TILE];
  // [-log2(e) lse 64 | delta 64] of the stage's queries; waves 2 and 3 repeat the two requests into the second half,
  // which nobody reads, so that the request sequence has no branch and can be issued between MFMAs
  __shared__ __attribute__((aligned(256))) float stat0[4 * BQ];
  __shared__ __attribute__((aligned(256))) float stat1[4 * BQ];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), hf = lane >> 5, jl = lane & 31;
  int row, jt;                                    // key tile 0 is seen by the most queries: heaviest first
  map_block(blockIdx.x, a.G * a.B, row, jt);
  int chunk = 0;
  // (chunk by chunk over all tiles: the workgroups that run together then share the query tiles of the same heads in L2)
  if (SPLIT) { const int ntile = (a.L + BJ - 1) / BJ; chunk = jt / ntile; jt %= ntile; }
  const int g = row % a.G, b = row / a.G;
  const int rep = a.H / a.G;
  const int j0 = jt * BJ, jw0 = j0 + wave * 32, j = jw0 + jl;
  const SeqView sv = seq_view(a, b);
  if (j0 >= sv.L) return;                         // packed batch: this entry is shorter than the longest one
  const bool j_ok = j < sv.L;
  const int jc = j_ok ? j : sv.L - 1;
  const int64_t kvrow = ((sv.kv0 + jc) * a.G + g) * HD;
  const bf16_t* Kg = (const bf16_t*)a.k + kvrow;
  const bf16_t* Vg = (const bf16_t*)a.v + kvrow;
  const int64_t qs = (int64_t)a.H * HD;

  // This lane's K and V rows are requested before any of the mask's arithmetic, the first Q / dO tile as soon as the
  // first query tile is known, and the rest of that arithmetic (three more integer divisions) runs while they travel.
  bf16x8_t kf[8], vf[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    kf[s] = *(const bf16x8_t*)(Kg + 16 * s + 8 * hf);
    vf[s] = *(const bf16x8_t*)(Vg + 16 * s + 8 * hf);
  }
  __builtin_amdgcn_sched_barrier(0);

  // first query that sees any key of the workgroup; below: this lane's key / any key of the wave / every key of the wave
  const MaskParams mk = sample_mask(a, b);
  const int wg_first = first_query_seeing(j0, mk);
  const int qt0 = wg_first / BQ;
  const int nqt = (sv.S + BQ - 1) / BQ;
  const int per_head = nqt > qt0 ? nqt - qt0 : 0;
  int iters = per_head * rep;                       // (head, query tile) pairs, head-major
  int first = 0;                                    // this workgroup's first
  bool whole = true;                                // no other workgroup shares the key tile
  if (SPLIT) {
    whole = tile_chunks(iters, sp.per_chunk) == 1;
    first = chunk * sp.per_chunk;
    if (chunk > 0 && first >= iters) return;
    iters = min(iters - first, sp.per_chunk);
  }
  int fq, wave_first, wave_all;                     // set behind the first tile's requests
  const float c2 = a.scale * LOG2E;
  const FragOffs fo = make_frag_offs(lane);

  // In accumulation registers by hand (mfma_in_place), with the scores in vector registers: the compiler keeps all of a function's
  // accumulators in one register file.  With all in the one, the scores' 64 values were copied in every tile (2689 -> 2648 us for
  // 2 x 4096 positions in 8 groups, 6684 -> 6566 for 8192 at 5120 channels); with all in the other, one LDS fragment was in flight
  // instead of four.
  f32x16_t dk[4], dv[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) { dk[i][e] = 0.f; dv[i][e] = 0.f; }

  // Q / dO rows and the LSE / delta entries of tile `it`; rows and entries past
  // the sequence end arrive as zeros (zero Q and dO rows contribute nothing).
  int f_hh = 0, f_qt = qt0;                         // fetch cursor: head within the group, query tile
  if (SPLIT && first > 0) { f_hh = first / per_head; f_qt = qt0 + first % per_head; }
  int c_qt = f_qt;                                  // compute cursor: query tile
  const int64_t head0 = sv.q0 * a.H + g * rep + f_hh;
  const bf16_t* f_q = (const bf16_t*)a.q + head0 * HD;           // row 0 of the fetch cursor's head
  const bf16_t* f_do = (const bf16_t*)a.dout + head0 * HD;
  const float* f_stat = ((wave & 1) == 0 ? a.nlse2 : a.delta) + sv.lse0 + (g * rep + f_hh) * sv.lse_hs;
  const int tile_bytes = sv.S > 0 ? (int)((((int64_t)sv.S - 1) * qs + HD) * 2) : 0;   // one head's Q (dO) rows of this entry
  // request i of 9, in order; the cursor moves on behind the last one
  auto fetch_part = [&](int i, bf16_t* st, float* stat) BEAGLE_INLINE_LAMBDA {
    const int q0 = f_qt * BQ;
    const bool live = f_hh < rep;                    // past the last pair: empty descriptors, i.e. zeros
    if (i < 4) load_rows_part(st, __builtin_amdgcn_make_buffer_rsrc((void*)f_q, 0, live ? tile_bytes : 0, 0x00020000), qs, q0, tid, i);
    else if (i < 8)
      load_rows_part(st + TILE, __builtin_amdgcn_make_buffer_rsrc((void*)f_do, 0, live ? tile_bytes : 0, 0x00020000), qs, q0, tid, i - 4);
    else {
      const __amdgpu_buffer_rsrc_t srs = __builtin_amdgcn_make_buffer_rsrc((void*)f_stat, 0, live ? sv.S * 4 : 0, 0x00020000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(srs, (lds_void_ptr)(stat + wave * BQ), 4, (q0 + lane) * 4, 0, 0, 0);
      // advance the cursor without branches
      const bool wrap = f_qt + 1 == nqt;
      const bool adv = wrap && f_hh + 1 < rep;
      f_qt = wrap ? qt0 : f_qt + 1;
      f_hh += wrap ? 1 : 0;
      f_q += adv ? HD : 0; f_do += adv ? HD : 0; f_stat += adv ? sv.lse_hs : 0;
    }
  };
  auto fetch = [&](bf16_t* st, float* stat) {
#pragma unroll
    for (int i = 0; i < 9; ++i) fetch_part(i, st, stat);
  };

  auto tile_step = [&](const bf16_t* cur, const float* sl, bf16_t* nxt, float* nstat) {
    const int q0 = c_qt * BQ;
    if (++c_qt == nqt) c_qt = qt0;
    if (q0 + BQ <= wave_first) fetch(nxt, nstat);     // a wave that sees nothing of the tile only requests its share of the next
    if (q0 + BQ > wave_first) {                       // some query of the tile sees some key of the wave
      const bf16_t* qsm = cur;
      const bf16_t* dsm = cur + TILE;
      const int relq = fq - q0 - 4 * hf;    // query offsets inside the tile are compile-time constants
      // The tile is one run of 64 MFMAs: the scores (S and dP in turn) of its first block of 32 queries, those of the second, then
      // either's accumulation (dV and dK in turn).  A step is an MFMA and its share of everything else: the read of the LDS fragment
      // that the MFMA four further on wants, the next tile's requests, the statistics' reads, and, one phase late, the probabilities
      // and products of a block, two elements at a time.  A fence at its end keeps it apart from the next one; inside a step the
      // order is the compiler's (a block's first probabilities stand ahead of their step's MFMA and wait for S, two MFMAs back).
      // This kernel has one wave per SIMD: whatever is not in its place leaves the matrix pipe idle, and every phase that started
      // with reads of its own did.  Training steps against phases in the compiler's order, us: 4096 positions in 8 groups x 2 2600 ->
      // 2571, 8192 at 5120 channels 6454 -> 6327; six or eight fragments ahead measure the same.
      // Register e of block qb is query q0 + 32 qb + 8 (e/4) + 4 hf + e%4 ; column = this lane's key.
      f32x16_t s2[2], dp[2];
      float4 l4[2][4], d4[2][4];
      float pv[2][16];
      union probs_t { uint32_t u[4]; bf16x8_t v; } pp[2][2], pd[2][2];
      bf16x8_t fr[64];
      auto read = [&](int n) BEAGLE_INLINE_LAMBDA {
        const bf16_t* t = n & 1 ? (n < 32 ? dsm : qsm) : (n < 32 ? qsm : dsm);
        if (n < 32) fr[n] = row_frag(t, fo, n >> 4, (n >> 1) & 7);
        else fr[n] = tr_frag(t, fo, 2 * (n - 32) & ~15, (n >> 1) & 3);
      };
      auto mfma = [&](int n) BEAGLE_INLINE_LAMBDA {
        const int i = n >> 1, qb = (n >> 4) & 1;
        if (n < 32) {
          f32x16_t& c = n & 1 ? dp[qb] : s2[qb];
          if ((i & 7) == 0)
#pragma unroll
            for (int e = 0; e < 16; ++e) c[e] = 0.f;
          c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[n], n & 1 ? vf[i & 7] : kf[i & 7], c, 0, 0, 0);
        } else {
          const int t = (n >> 3) & 1;
          mfma_in_place(n & 1 ? dk[i & 3] : dv[i & 3], fr[n], n & 1 ? pd[qb][t].v : pp[qb][t].v);
        }
      };
      auto stat = [&](int qb, int i) BEAGLE_INLINE_LAMBDA {
        const int r = 32 * qb + 8 * (i & 3) + 4 * hf;
        if (i < 4) l4[qb][i] = *(const float4*)(sl + r);
        else d4[qb][i & 3] = *(const float4*)(sl + BQ + r);
      };
      auto probs = [&](int qb, int m) BEAGLE_INLINE_LAMBDA {        // m: 0 .. 7 probabilities, 8 .. 15 products
        const int e = 2 * (m & 7);
        if (m < 8) {
          const float* ls = (const float*)&l4[qb][e >> 2];
          pv[qb][e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s2[qb][e], c2, ls[e & 3]));
          pv[qb][e + 1] = __builtin_amdgcn_exp2f(__builtin_fmaf(s2[qb][e + 1], c2, ls[(e & 3) + 1]));
          // The per-element predicate only where some key of the wave is hidden from some query of the block (a
          // scalar branch around the compares and selects alone: the kernel is bound by instruction issue, and a
          // second copy of the whole body made the register allocator shuffle the accumulators).  A blind query
          // (-log2(e) LSE = +inf, p = +inf) is below fq for every key, so its block always comes through here.
          if (m == 7 && q0 + 32 * qb < wave_all) {
#pragma unroll
            for (int k = 0; k < 16; ++k)
              if (32 * qb + 8 * (k >> 2) + (k & 3) < relq) pv[qb][k] = 0.f;
          }
        } else {
          const float* dl = (const float*)&d4[qb][e >> 2];
          const float a0 = pv[qb][e], a1 = pv[qb][e + 1];
          pp[qb][e >> 3].u[(e >> 1) & 3] = cvt_pk(a0, a1);
          pd[qb][e >> 3].u[(e >> 1) & 3] = cvt_pk(a0 * (dp[qb][e] - dl[e & 3]), a1 * (dp[qb][e + 1] - dl[(e & 3) + 1]));
          // (here and not where they are used, which mfma_in_place would not wait for)
          if ((m & 3) == 3) asm volatile("" : "+v"(pp[qb][e >> 3].v), "+v"(pd[qb][e >> 3].v));
        }
      };
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int n = 0; n < AHEAD; ++n) read(n);
      __builtin_amdgcn_sched_barrier(0);
      static_for<0, 64>([&](auto n_) BEAGLE_INLINE_LAMBDA {
        constexpr int n = decltype(n_)::value;
        mfma(n);
        if constexpr (n + AHEAD < 64) read(n + AHEAD);
        if constexpr (n < 9) fetch_part(n, nxt, nstat);
        if constexpr (n >= 8 && n < 16) stat(0, n - 8);
        if constexpr (n >= 24 && n < 32) stat(1, n - 24);
        if constexpr (n >= 16 && n < 32) probs(0, n - 16);
        if constexpr (n >= 32 && n < 48) probs(1, n - 32);
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    wait_vmem();
    __syncthreads();
  };

  if (iters > 0) fetch(stage0, stat0);
  __builtin_amdgcn_sched_barrier(0);
  fq = j_ok ? first_query_seeing(j, mk) : sv.S;
  wave_first = jw0 < sv.L ? first_query_seeing(jw0, mk) : sv.S;
  wave_all = jw0 < sv.L ? first_query_seeing(min(jw0 + 32, sv.L) - 1, mk) : sv.S;
  __builtin_amdgcn_sched_barrier(0);
  wait_vmem();
  __syncthreads();
  int it = 0;
#pragma unroll 1
  for (; it + 2 <= iters; it += 2) {
    tile_step(stage0, stat0, stage1, stat1);
    tile_step(stage1, stat1, stage0, stat0);
  }
  if (it < iters) tile_step(stage0, stat0, stage1, stat1);
  mfma_drain();

  if (SPLIT && !whole) {
    // a share of the sums: as the accumulators lie, 1 KB per store instruction; sum_dkv_kernel adds the shares in order
    float* slot = sp.part + (((int64_t)row * ((a.L + BJ - 1) / BJ) + jt) * sp.chunks + chunk) * SLOT + wave * 4096 + lane * 4;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        *(float4*)(slot + (4 * cb + qd) * 256) = float4{dk[cb][4 * qd], dk[cb][4 * qd + 1], dk[cb][4 * qd + 2], dk[cb][4 * qd + 3]};
        *(float4*)(slot + BJ * HD + (4 * cb + qd) * 256) = float4{dv[cb][4 * qd], dv[cb][4 * qd + 1], dv[cb][4 * qd + 2], dv[cb][4 * qd + 3]};
      }
    return;
  }
  // ---- dK, dV rows out, through LDS (both stages are free: the last step ended with the requests landed and a barrier)
  {
    uint2 pk[16], pv[16];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        pk[4 * cb + qd] = make_uint2(cvt_pk(dk[cb][4 * qd] * a.scale, dk[cb][4 * qd + 1] * a.scale),
                                     cvt_pk(dk[cb][4 * qd + 2] * a.scale, dk[cb][4 * qd + 3] * a.scale));
        pv[4 * cb + qd] = make_uint2(cvt_pk(dv[cb][4 * qd], dv[cb][4 * qd + 1]), cvt_pk(dv[cb][4 * qd + 2], dv[cb][4 * qd + 3]));
      }
    const int64_t wrow = ((sv.kv0 + jw0) * a.G + g) * HD;               // row of the wave's first key
    const int64_t kvs = (int64_t)a.G * HD;
    store_rows_via_lds(stage0 + wave * 32 * HD, pk, lane, (bf16_t*)a.dk + wrow, kvs, sv.L - jw0);
    store_rows_via_lds(stage1 + wave * 32 * HD, pv, lane, (bf16_t*)a.dv + wrow, kvs, sv.L - jw0);
  }
}

// dK, dV of the key tiles that several workgroups shared: the sum of their shares, in chunk order.  One workgroup per
// (32 keys of a tile, matrix): 16 KB per share, summed as they lie, turned into rows in LDS.
__global__ __launch_bounds__(256) void sum_dkv_kernel(AttnArgs a, dkv::Split sp) {
  using namespace dkv;
  __shared__ __attribute__((aligned(16))) bf16_t rows[32][HD + 8];
  const int tid = threadIdx.x, ntile = (a.L + BJ - 1) / BJ;
  const int w = blockIdx.x & 3, mat = (blockIdx.x >> 2) & 1, tile = blockIdx.x >> 3;
  const int jt = tile % ntile, row = tile / ntile, g = row % a.G, b = row / a.G;
  const SeqView sv = seq_view(a, b);
  const int j0 = jt * BJ, jw0 = j0 + 32 * w;
  if (jw0 >= sv.L) return;
  const int n = tile_chunks(tile_pairs(j0, sample_mask(a, b), sv.S, a.H / a.G), sp.per_chunk);
  if (n == 1) return;
  const float* src = sp.part + (int64_t)tile * sp.chunks * SLOT + mat * BJ * HD + w * 4096;
  const float scale = mat == 0 ? a.scale : 1.f;
  float4 acc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i] = float4{0.f, 0.f, 0.f, 0.f};
  for (int c0 = 0; c0 < n; c0 += 4) {                // four shares (16 loads) in flight; past the last one: it again, unused
    float4 t[4][4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) t[c][i] = *(const float4*)(src + (int64_t)min(c0 + c, n - 1) * SLOT + (tid + 256 * i) * 4);
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (c0 + c < n) {
#pragma unroll
        for (int i = 0; i < 4; ++i) { acc[i].x += t[c][i].x; acc[i].y += t[c][i].y; acc[i].z += t[c][i].z; acc[i].w += t[c][i].w; }
      }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int idx = tid + 256 * i, piece = idx >> 6, lane = idx & 63;
    *(uint2*)&rows[lane & 31][8 * piece + 4 * (lane >> 5)] =
        make_uint2(cvt_pk(acc[i].x * scale, acc[i].y * scale), cvt_pk(acc[i].z * scale, acc[i].w * scale));
  }
  __syncthreads();
  bf16_t* out = (bf16_t*)(mat == 0 ? a.dk : a.dv) + ((sv.kv0 + jw0) * a.G + g) * HD;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int idx = tid + 256 * i, r = idx >> 4, c = idx & 15;
    if (jw0 + r < sv.L) *(uint4*)(out + (int64_t)r * a.G * HD + 8 * c) = *(const uint4*)&rows[r][8 * c];
  }
}

// Workgroups of the dK/dV kernel per key tile.  A tile's pairs are one serial chain of 1.9 us each; under grouped-query
// attention the heads of a group multiply it, and a short batch ends up with a few long chains on a few CUs.  With up to
// 256 tiles (one workgroup per CU) the chains are cut so that about one round of workgroups has work: tiles are seen by
// half of the queries on average, so n chunks make tiles (n + 1) / 2 of them.  Measured with 32 heads in 8 groups, us, one
// workgroup per tile -> n chunks + their sum: 300 positions (24 tiles) 42 -> 23, 777 (56) 93 -> 38, 1300 (88) 144 -> 60, 2048
// (128) 222 -> 106, 4096 (256) 448 -> 332.  Beyond that the shares cost what the balance gains (5546: 636 -> 614 at best, 8192:
// 574 -> 608), and so they do where the chain is short (777 positions, 32 groups: 34 -> 39).  Fewer where the caller's
// workspace has no room for as many shares, down to none.
static int64_t dkv_chunks(int64_t tiles, int64_t longest, int64_t most) {
  if (tiles > 256) return 1;
  int64_t n = tiles > 128 ? 2 : (448 + tiles / 2) / tiles - 1;
  if (n > 16) n = 16;
  if (n > most) n = most;
  return n > 1 && longest - (longest + n - 1) / n >= 10 ? n : 1;
}
static int64_t dkv_tiles(const AttnArgs& a) { return (int64_t)((a.L + dkv::BJ - 1) / dkv::BJ) * a.G * a.B; }
static int64_t dkv_longest(const AttnArgs& a) { return (int64_t)((a.S + dkv::BQ - 1) / dkv::BQ) * (a.H / a.G); }
constexpr size_t SHARE_BYTES = dkv::SLOT * sizeof(float);
static dkv::Split dkv_split(const AttnArgs& a, void* shares, size_t share_bytes) {
  const int64_t tiles = dkv_tiles(a), longest = dkv_longest(a);
  const int64_t n = dkv_chunks(tiles, longest, (int64_t)(share_bytes / (tiles * SHARE_BYTES)));
  if (n == 1) return {nullptr, 1, 0x7fffffff};
  const int64_t per = (longest + n - 1) / n;
  return {(float*)shares, (int32_t)((longest + per - 1) / per), (int32_t)per};
}

// workspace: the pre-scaled LSE array, as large as delta
size_t attn_bwd_bf16_ws_bytes(const AttnArgs& a) { return (size_t)a.B * a.H * a.S * sizeof(float); }
// ... and what the shares of split key tiles take at most, for this problem or any that is no larger in batch and lengths
// (of equal lengths if this one's are): a program that sizes its workspace by its largest batch has the smaller ones split too
size_t attn_bwd_bf16_share_bytes(const AttnArgs& a) {
  const int64_t ltiles = (a.L + dkv::BJ - 1) / dkv::BJ, rep = a.H / a.G, all = dkv_longest(a);
  int64_t n = 0;
  for (int64_t u = 1; u * a.G <= 256 && u <= ltiles * a.B; ++u) {      // key tiles per group
    const int64_t own = (u < ltiles ? u : ltiles) * (dkv::BJ / dkv::BQ) * rep;
    const int64_t c = dkv_chunks(u * a.G, a.S == a.L && own < all ? own : all, 16);
    if (c > 1 && u * a.G * c > n) n = u * a.G * c;
  }
  return (size_t)n * SHARE_BYTES;
}

void launch_attn_bwd_bf16(const AttnArgs& args, void* ws, void* shares, size_t share_bytes, hipStream_t s) {
  AttnArgs a = args;
  a.nlse2 = (float*)ws;
  {
    ProfScope ps("attn_bwd_dq_bf16", s);
    if (attn_key_halves(a)) hipLaunchKernelGGL(attn_bwd_dq_bf16_kernel<2>, dim3((a.S + 63) / 64 * a.H * a.B), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(attn_bwd_dq_bf16_kernel<1>, dim3((a.S + 127) / 128 * a.H * a.B), dim3(256), 0, s, a);
  }
  const dkv::Split sp = dkv_split(a, shares, share_bytes);
  const int tiles = (int)dkv_tiles(a);
  {
    ProfScope ps("attn_bwd_dkv_bf16", s);
    if (sp.chunks > 1) hipLaunchKernelGGL(attn_bwd_dkv_bf16_kernel<true>, dim3(tiles * sp.chunks), dim3(256), 0, s, a, sp);
    else hipLaunchKernelGGL(attn_bwd_dkv_bf16_kernel<false>, dim3(tiles), dim3(256), 0, s, a, sp);
  }
  if (sp.chunks > 1) {
    ProfScope ps("attn_bwd_dkv_sum", s);
    hipLaunchKernelGGL(sum_dkv_kernel, dim3(tiles * 8), dim3(256), 0, s, a, sp);
  }
}

}  // namespace beagle
