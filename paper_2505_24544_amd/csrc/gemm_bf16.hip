// bf16 GEMM on the gfx950 matrix cores: C[M,N] = X * W (+ X2 * W2), float
// accumulation, for the Q/K/V/output projections of Eq. 2 and every
// projection-shaped contraction of the backward pass.
//
// Design
//   * One workgroup of 4 wavefronts (2 x 2) owns a 256 x 256 tile of C (128 x
//     128 for shallow products); each wave owns a quarter of it as accumulators
//     of v_mfma_f32_16x16x32_bf16, which the power limit lets run 6 % faster on
//     random operands than 32x32x16 (bare loops: 1.90 against 1.80 PFLOP/s; it
//     reads and writes half the accumulators per product).
//   * The k loop walks 32 k at a time.  Slices go from HBM/L2 straight into LDS
//     (buffer_load ... lds, 16 bytes per lane): no staging registers, no
//     ds_write, and out-of-range chunks arrive as zeros through the buffer
//     descriptor's range check.
//   * What bounded it was the trip to memory: two stages of 64 k left a request
//     1000 - 2000 cycles, and a slice of 64 k took 2900 - 3300 cycles with loads
//     from memory, 2340 with loads that always hit L2, 2048 of MFMAs.  All 160 KB
//     of LDS now hold stages, each is requested anew as soon as every wave has
//     its fragments, and the requests are spread evenly over the MFMAs: 2000 -
//     4000 cycles from request to use, 2240 - 2380 cycles per 64 k.
//   * k-contiguous operands are requested 64 k (a 128-byte line) at a time: by
//     halves of lines L2 served twice the requests, and X * W^T took 2900 cycles
//     per 64 k instead of 2290.  Row-contiguous ones come 32 k at a time.
//   * Each operand tile sits in LDS in the order it has in HBM (a lane's 16
//     bytes land at wave_base + 16 * lane), with an XOR swizzle chosen on the
//     GLOBAL side (which chunk a lane fetches) so that reads are conflict free:
//     a k-contiguous fragment is one ds_read_b128, a row-contiguous one two
//     ds_read_b64_tr_b16 (the LDS transpose read), which hand every lane four
//     consecutive k of its own row.
//   * Fragments are double-buffered in registers: those of the next step are
//     read from LDS between the MFMAs of this one.  Reads, requests and scalar
//     arithmetic each have their place behind an MFMA; one barrier per step.
//   * The MFMA is issued "transposed" (A operand = W rows, B operand = X rows)
//     so that a lane ends up with 4 consecutive n of one C row in 4 consecutive
//     accumulator registers.
//   * Workgroup ids are remapped so that each XCD (ids are dealt round-robin
//     to the 8 XCDs) works on a contiguous run of tiles, and tiles are walked
//     in groups of GROUP_M tile-rows so that the run shares X and W tiles in
//     that XCD's L2.
//   * Several independent GEMMs can share one launch (Q, K, V projections;
//     the three weight gradients) so that small ones do not leave CUs idle.
// Measured against the kernel of two stages and 32x32x16 MFMAs, us (operands in
// HBM): 8192 x 4096 x 4096 X W 211 -> 187, X W^T 221 -> 183, X^T Y over 8192 k 204 ->
// 181; 3048 x 4096 x 11008 (192 tiles) 262 -> 214.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include "common.h"
#include "mfma_in_place.h"

namespace beagle {

typedef mfma_bf16x8_t bf16x8_t;
typedef mfma_f32x16_t f32x16_t;
typedef mfma_f32x4_t f32x4_t;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4_t;
typedef s16x4_t __attribute__((address_space(3))) * lds_s16x4_ptr;
typedef __attribute__((address_space(3))) void* lds_void_ptr;
// Where a tile's rows go.  The type says that it is global memory: a generic pointer that an empty asm has hidden becomes flat stores,
// which the LDS counter covers too, so that every wait for a patch waits for the stores in front of it.  (Up to 0.4 % of a call: 1013
// states into the cache 69.7 / 69.5 us, a step of 777 rows 323.8 / 323.1.)
typedef unsigned int out_u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) char* out_ptr;
typedef __attribute__((address_space(1))) out_u32x4* out_u32x4_ptr;

constexpr int BK = 64;
constexpr int KB = 32;                               // k per step of gemm_bf16_kernel
constexpr int GROUP_M = 4;
constexpr int NUM_XCD = 8;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)bytes, 0x00020000);
}

// 16 bytes per lane, HBM/L2 -> LDS at dst + 16 * lane
__device__ __forceinline__ void request16(__amdgpu_buffer_rsrc_t rsrc, bf16_t* dst, int off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)dst, 16, off, 0, 0, 0);
}

// Tiles of operands whose rows are contiguous: chunk c of k-row k sits at chunk c ^ krow_swizzle(k).  (Of k-contiguous ones, 128 bytes
// per row: chunk c of row r at chunk c ^ ((r >> 1) & 7).)
__device__ __forceinline__ int krow_swizzle(int k) { return ((k & 3) << 2) ^ ((k >> 2) & 2); }
// Where the requests of one operand stand: a slice of both k segments after the other.  The descriptor starts at the current slice,
// so the lanes' offsets are constants of the tile and a slice costs scalar arithmetic only, in pieces that fit between two MFMAs;
// past the last slice it is empty.
struct SliceCursor {
  const char *at, *at2;                              // the slice's first byte for this tile; the second segment's
  int left, left2, step;                             // bytes from there to the operand's end; bytes per slice
  int t, sw, end;                                    // the slice's number; the number at which the operand changes; of slices
  bf16_t *first, *dst;                               // where this wave's part of stage 0 lies, and of the slice's stage
  __amdgpu_buffer_rsrc_t rsrc;
  static constexpr int PIECES = 4;

  // operand (p, then p2) of `rows` rows, tile from row r0, k per slice
  __device__ __forceinline__ void init(const GemmArgs& g, const void* p, const void* p2, bool kmajor, int rows, int r0, int ld, int k, bf16_t* stage0) {
    const int64_t skip = (kmajor ? (int64_t)r0 * ld : (int64_t)r0) * 2;
    at = (const char*)p + skip; at2 = (const char*)p2 + skip;
    left = (int)((int64_t)(kmajor ? rows : g.K) * ld * 2 - skip); left2 = (int)((int64_t)(kmajor ? rows : g.K2) * ld * 2 - skip);
    step = kmajor ? k * 2 : k * ld * 2;
    t = 0; sw = (g.K + k - 1) / k; end = sw + (p2 ? (g.K2 + k - 1) / k : 0);
    first = dst = stage0;
    // (in registers: the loop would fetch what it can from the arguments again, and wait for it)
    asm volatile("" : "+s"(at2), "+s"(left2), "+s"(step), "+s"(end));
    if (sw == 0) { at = at2; left = left2; sw = end; }
    if (end == 0) left = 0;
  }
  __device__ __forceinline__ void describe() { rsrc = make_rsrc(at, max(left, 0)); }
  // on to the next slice: pieces 0 .. PIECES - 1 in order; STAGES stages of E elements
  template <int I, int STAGES, int E> __device__ __forceinline__ void next() {
    if constexpr (I == 0) { at += step; left -= step; }
    if constexpr (I == 1) dst = dst == first + (STAGES - 1) * E ? first : dst + E;
    if constexpr (I == 2) {
      if (++t == sw) {                               // on to the second segment, or past the end: nothing left
        at = at2;
        left = t < end ? left2 : 0;
        sw = t < end ? end : -1;
      }
    }
    if constexpr (I == 3) describe();
  }
};

// Workgroup id -> (problem, tile index inside the problem).  Ids are dealt
// round-robin to the 8 XCDs; every problem's tiles are split evenly over the
// XCDs (contiguous runs, so neighbouring tiles share an L2), and an XCD walks
// the problems in order.  Remainder tiles of successive problems go to
// successive XCDs, which keeps the per-XCD totals equal to what the hardware
// deals out.  Problems of different depth (dXkv has twice the k of dXq) are thus
// balanced across XCDs instead of being concentrated on some of them.
__device__ __forceinline__ void map_tile(int pid, const int* tiles, int count, int& prob, int& local) {
  const int c = pid % NUM_XCD;
  int idx = pid / NUM_XCD, off = 0;
  prob = count - 1; local = 0;
  for (int p = 0; p < count; ++p) {
    const int base = tiles[p] / NUM_XCD, rem = tiles[p] % NUM_XCD;
    const int r = (c - off + NUM_XCD) % NUM_XCD;
    const int cnt = base + (r < rem ? 1 : 0);
    if (idx < cnt || p + 1 == count) { prob = p; local = r * base + (r < rem ? r : rem) + idx; return; }
    idx -= cnt;
    off = (off + rem) % NUM_XCD;
  }
}

// Which tile of which problem a workgroup owns: map_tile, then tile rows in groups (of 1024 rows) so that the
// workgroups that run together share operand tiles in their XCD's L2.
template <int BM, int BN>
__device__ __forceinline__ void locate_tile(const GemmGroup& grp, int wg, int& prob, int& m0, int& n0) {
  constexpr int GROUP = GROUP_M * 256 / BM;
  int ntile[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    ntile[i] = i < grp.count ? ((grp.p[i].M + BM - 1) / BM) * ((grp.p[i].N + BN - 1) / BN) : 0;
  int pid;
  map_tile(wg, ntile, grp.count, prob, pid);
  const GemmArgs& g = grp.p[prob];
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  const int per_group = GROUP * tiles_n;
  const int first_m = (pid / per_group) * GROUP;
  const int gsz = min(tiles_m - first_m, GROUP);
  m0 = (first_m + (pid % per_group) % gsz) * BM;
  n0 = ((pid % per_group) / gsz) * BN;
}

// RES: some problem of the group has a residual operand R (a separate instantiation, so that the kernels
// without one keep their register allocation).
template <int T, bool XK, bool WK, bool F32OUT, bool RES>
__global__ __launch_bounds__(256, T == 4 ? 1 : 2) void gemm_bf16_kernel(GemmGroup grp) {
  static_assert(XK || !WK, "k-contiguous W comes with k-contiguous X");
  constexpr int NB = 2 * T;                          // 16 x 16 accumulators per wave: NB x NB
  constexpr int BM = 64 * T, BN = 64 * T;
  // steps of KB k per slice of X and of W, stages of either: 160 KB (T = 4) or 80 KB (T = 2) in all
  constexpr int XS = XK ? 2 : 1, WS = XK && WK ? 2 : 1, NXS = XK ? 3 : 5, NWS = WS == 2 ? 2 : XK ? 4 : 5;
  constexpr int AHEAD = XK ? 3 : 4;                  // steps from a step's requests to the barrier that wants them
  constexpr int XE = BM * KB * XS, WE = BN * KB * WS, WBASE = NXS * XE;      // elements per stage; where W's begin
  __shared__ __attribute__((aligned(1024))) bf16_t smem[NXS * XE + NWS * WE];

  int pi, m0, n0;
  locate_tile<BM, BN>(grp, blockIdx.x, pi, m0, n0);
  const GemmArgs& g = grp.p[pi];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave >> 1) * (32 * T), wn = (wave & 1) * (32 * T);

  f32x4_t acc[NB][NB];

  // ---- request side: for either operand a cursor over the slices of both k segments, and the lanes' offsets from there
  constexpr int XLD = BM * XS / 64, WLD = BN * WS / 64, NLD = XLD / XS + WLD / WS;      // requests per thread: an X slice, a W slice, a step
  const int ldx = (int)g.lda, ldw = (int)g.ldb;
  int nk = (g.K + KB - 1) / KB + (g.A2 ? (g.K2 + KB - 1) / KB : 0);           // steps
  auto chunk_off = [&](int q, bool kmajor, int rows, int ld) BEAGLE_INLINE_LAMBDA {      // 16-byte chunk q of an operand's slice
    if (kmajor) { const int r = q >> 3; return (r * ld + 8 * ((q & 7) ^ ((r >> 1) & 7))) * 2; }
    const int cpr = rows / 8, k = q / cpr;
    return (k * ld + 8 * ((q % cpr) ^ krow_swizzle(k))) * 2;
  };
  int xoff[XLD], woff[WLD];
#pragma unroll
  for (int i = 0; i < XLD; ++i) xoff[i] = chunk_off(tid + 256 * i, XK, BM, ldx);
#pragma unroll
  for (int i = 0; i < WLD; ++i) woff[i] = chunk_off(tid + 256 * i, WK, BN, ldw);
  SliceCursor fx, fw;
  fx.init(g, g.A, g.A2, XK, g.M, m0, ldx, KB * XS, smem + wave * 512);
  fw.init(g, g.B, g.B2, WK, g.N, n0, ldw, KB * WS, smem + WBASE + wave * 512);
  constexpr int PIECES = SliceCursor::PIECES;
  auto fx_next = [&](auto i_) BEAGLE_INLINE_LAMBDA { fx.next<decltype(i_)::value, NXS, XE>(); };
  auto fw_next = [&](auto i_) BEAGLE_INLINE_LAMBDA { fw.next<decltype(i_)::value, NWS, WE>(); };
  // Request i of a step.  X and W in turn where W's slices last a step; X's slices may last two, and are then requested half in an
  // odd step, half in the next one.  Where either's last two, X's in odd steps and W's in even ones.
  auto f_issue = [&](auto odd_, auto i_) BEAGLE_INLINE_LAMBDA {
    constexpr int i = decltype(i_)::value, odd = decltype(odd_)::value;
    constexpr bool of_w = WS == 2 ? !odd : i & 1;
    constexpr int n = WS == 2 ? i : (!of_w && XS == 2 && !odd ? XLD / 2 : 0) + (i >> 1);
    if constexpr (of_w) request16(fw.rsrc, fw.dst + n * 2048, woff[n]);
    else request16(fx.rsrc, fx.dst + n * 2048, xoff[n]);
  };

  // ---- fragment addresses (bytes) in the stages that are read next; everything else is an immediate
  typedef __attribute__((address_space(3))) bf16_t* lds_bf16_ptr;
  const int l16 = lane & 15, gi = lane >> 4;
  constexpr int NXA = XK ? XS : NB, NWA = WK ? WS : NB;       // one per step of a slice, or per block
  uint32_t xa[NXA], wa[NWA];
  {
    const uint32_t base = (uint32_t)(uintptr_t)(lds_bf16_ptr)smem;
    auto rows = [&](int r0, int b) BEAGLE_INLINE_LAMBDA { return ((r0 + l16) * KB * 2 + (((4 * b + gi) ^ ((l16 >> 1) & 7)) << 3)) * 2; };
    auto cols = [&](int rows, int r0, int b) BEAGLE_INLINE_LAMBDA {
      const int kr = 8 * gi + (l16 >> 2), col = r0 + 16 * b + 4 * (l16 & 3);
      return (kr * rows + ((((col >> 3) ^ krow_swizzle(kr)) << 3) | (col & 7))) * 2;
    };
#pragma unroll
    for (int b = 0; b < NXA; ++b) xa[b] = base + (XK ? rows(wm, b) : cols(BM, wm, b));
#pragma unroll
    for (int b = 0; b < NWA; ++b) wa[b] = base + 2 * WBASE + (WK ? rows(wn, b) : cols(BN, wn, b));
  }
  int rx_st = 0, rx_step = XE * 2, rw_st = 0, rw_step = WE * 2;     // the stage they point into; bytes from there to the next
  auto rx_next = [&]() BEAGLE_INLINE_LAMBDA { rx_st = rx_st + 1 == NXS ? 0 : rx_st + 1; rx_step = rx_st + 1 == NXS ? -(NXS - 1) * XE * 2 : XE * 2; };
  auto rw_next = [&]() BEAGLE_INLINE_LAMBDA { rw_st = rw_st + 1 == NWS ? 0 : rw_st + 1; rw_step = rw_st + 1 == NWS ? -(NWS - 1) * WE * 2 : WE * 2; };
  union frag_t { lds_u32x4_t u; struct { lds_u32x2_t a, b; } s; bf16x8_t v; };
  // Fragments, in buffers that take turns.  Where W's slices last two steps, both steps' fragments are read in the odd step before,
  // so that the stage is free a step earlier; three buffers, then, over a period of four steps.
  frag_t xf[2][NB], wf[WS == 2 ? 3 : 2][NB];
  constexpr int PERIOD = WS == 2 ? 4 : 2;
  // LDS read n of step P of a period, X fragments first (one read each, or two transpose reads), then W's; behind the last read of
  // an address, it moves on to the next stage
  constexpr int NXR = XK ? NB : 2 * NB, NWR = WK ? NB : 2 * NB;
  auto wbuf = [](int p) constexpr { return WS == 1 ? p % 2 : p % 2 == 0 ? 0 : p % 4 == 1 ? 1 : 2; };
  auto read_one = [&](auto p_, auto n_) BEAGLE_INLINE_LAMBDA {
    constexpr int nxt = decltype(p_)::value + 1, n = decltype(n_)::value, fx_ = nxt % 2;
    if constexpr (n < NXR) {
      if constexpr (XK) lds_read_b128<n * 16 * KB * XS * 2>(xf[fx_][n].u, xa[fx_]);
      else if constexpr (n & 1) lds_read_tr16_b64<4 * BM * 2>(xf[fx_][n >> 1].s.b, xa[n >> 1]);
      else lds_read_tr16_b64<0>(xf[fx_][n >> 1].s.a, xa[n >> 1]);
      if constexpr (XK ? n == NXR - 1 : n & 1) xa[XK ? fx_ : n >> 1] += rx_step;
    } else {
      constexpr int half = (n - NXR) / NWR, k = (n - NXR) % NWR, fw_ = wbuf(nxt + half);
      if constexpr (WK) lds_read_b128<k * 16 * KB * WS * 2>(wf[fw_][k].u, wa[half]);
      else if constexpr (k & 1) lds_read_tr16_b64<4 * BN * 2>(wf[fw_][k >> 1].s.b, wa[k >> 1]);
      else lds_read_tr16_b64<0>(wf[fw_][k >> 1].s.a, wa[k >> 1]);
      if constexpr (WK ? k == NWR - 1 : k & 1) wa[WK ? half : k >> 1] += rw_step;
    }
  };
  auto frags_wait = [&](auto p_) BEAGLE_INLINE_LAMBDA {                   // what step P read is in registers; nothing that uses it moves up
    constexpr int nxt = decltype(p_)::value + 1;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      lds_tie(xf[nxt % 2][i].u);
      if (WS == 1 || nxt % 2 == 0) lds_tie(wf[wbuf(nxt)][i].u);
      if (WS == 2 && nxt % 2 == 0) lds_tie(wf[wbuf(nxt + 1)][i].u);
    }
  };
  auto landed = [&](auto n_) BEAGLE_INLINE_LAMBDA {                       // all but the requests of the n youngest steps have landed, for every wave
    constexpr int n = decltype(n_)::value * NLD;
    __builtin_amdgcn_s_waitcnt((n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // Step P of a period, KB k; on entry its fragments are in registers.  Behind the barrier the next step's operands are visible and
  // every wave has this step's fragments, so the stages they came from are requested anew, two or three steps (of 1024 cycles of
  // MFMAs) before they are waited for.  Every MFMA is pinned in its place, with at most one read, one request or one piece of a
  // cursor's arithmetic behind it.
  auto step = [&](auto p_) BEAGLE_INLINE_LAMBDA {
    constexpr int P = decltype(p_)::value, odd = P & 1;
    constexpr int NM = NB * NB, RE = NM / NLD;       // MFMAs, per request
    constexpr int NR = NXR + (WS == 1 ? NWR : odd ? 2 * NWR : 0);
    constexpr bool XEND = XS == 1 || (WS == 2 ? odd : !odd), WEND = WS == 1 || !odd;      // this step's requests end a slice
    constexpr bool XREAD = XS == 1 || !odd, WREAD = WS == 1 || odd;                       // its reads do
    if constexpr (WS == 1 || odd) landed(int_c<AHEAD - 1>{});
    else __builtin_amdgcn_s_barrier();               // (an even step reads from slices that the odd one has waited for)
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NM>([&](auto m_) BEAGLE_INLINE_LAMBDA {
      constexpr int m = decltype(m_)::value, i = m / NB, j = (i & 1) ? NB - 1 - m % NB : m % NB;
      mfma_in_place(acc[i][j], wf[wbuf(P)][j].v, xf[odd][i].v);
      constexpr int r0 = m * NR * 5 / (NM * 4), r1 = (m + 1) * NR * 5 / (NM * 4);      // reads behind the first four fifths
      if constexpr (r0 < NR) static_for<r0, (r1 < NR ? r1 : NR)>([&](auto n_) BEAGLE_INLINE_LAMBDA { read_one(p_, n_); });
      if constexpr (m % RE == 0) f_issue(int_c<odd>{}, int_c<m / RE>{});
      if constexpr (T == 4) {
        constexpr int px = m - (NM - (WS == 2 ? 1 : 2) * RE + 1), pw = m - (NM - RE + 1);
        if constexpr (XEND && px >= 0 && px < PIECES) fx_next(int_c<px>{});
        if constexpr (WEND && pw >= 0 && pw < PIECES) fw_next(int_c<pw>{});
        if constexpr (XREAD && pw == PIECES) rx_next();
        if constexpr (WREAD && pw == PIECES + 1) rw_next();
      } else if constexpr (m == NM - 1) {
        if constexpr (XEND) static_for<0, PIECES>(fx_next);
        if constexpr (WEND) static_for<0, PIECES>(fw_next);
        if constexpr (XREAD) rx_next();
        if constexpr (WREAD) rw_next();
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    frags_wait(p_);
  };

  // the requests of the steps that would have been: AHEAD, and before them the one that brings X's first (half) slice
  fx.describe(); fw.describe();
  auto before = [&](auto odd_, auto with_w_) BEAGLE_INLINE_LAMBDA {
    constexpr int odd = decltype(odd_)::value;
    constexpr bool with_w = decltype(with_w_)::value;
    static_for<0, NLD>([&](auto i_) BEAGLE_INLINE_LAMBDA { if constexpr (with_w || !(decltype(i_)::value & 1)) f_issue(odd_, i_); });
    if constexpr (XS == 1 || (WS == 2 ? odd : !odd)) static_for<0, PIECES>(fx_next);
    if constexpr (WS == 2 ? !odd : with_w) static_for<0, PIECES>(fw_next);
  };
  if constexpr (XS == 2) before(int_c<1>{}, int_c<(WS == 2)>{});
  static_for<0, AHEAD + 1>([&](auto t_) BEAGLE_INLINE_LAMBDA { before(int_c<(decltype(t_)::value & 1)>{}, int_c<1>{}); });
  __builtin_amdgcn_sched_barrier(0);
  // (cleared behind the first requests, not ahead of them: 256 register writes per lane are 2 000 cycles that the trip hides)
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;
  __builtin_amdgcn_sched_barrier(0);
  landed(int_c<AHEAD>{});
  static_for<0, NXR + WS * NWR>([&](auto n_) BEAGLE_INLINE_LAMBDA { read_one(int_c<PERIOD - 1>{}, n_); });
  if constexpr (XS == 1) rx_next();
  rw_next();
  frags_wait(int_c<PERIOD - 1>{});
  int kt = 0;
#pragma unroll 1
  for (; kt + PERIOD <= nk; kt += PERIOD) static_for<0, PERIOD>(step);
  // (k-contiguous operands come in whole slices of BK)
  if constexpr (WS == 2) { if (kt < nk) { step(int_c<0>{}); step(int_c<1>{}); } }
  if constexpr (!XK) { if (kt < nk) step(int_c<0>{}); }
  mfma_drain();
  __builtin_amdgcn_s_waitcnt(0x0F70);                // the requests past the end (they write zeros) have landed
  __builtin_amdgcn_sched_barrier(0);

  // ---- epilogue: lane holds C row m = .. + lane % 16; register e of tile (i, j) holds column n = .. + 4 * (lane / 16) + e.
  // Straight from the registers a store instruction would carry 8 (float: 64) bytes for each of 64 (16) places, and the workgroup --
  // the only one on its CU -- spent 15 % of its life issuing them (27 500 cycles per 256 x 256 tile of bf16 against 2 300 per 64 k).
  // Each wave therefore transposes its part of the tile through a patch of LDS of its own and writes whole row segments, 16
  // bytes per lane.  Patch rows are made of 16-byte chunks; chunk c of row r sits at position c ^ (r % chunks), which spreads the
  // column-wise writes over the banks.
  // (the bounds in registers: otherwise every one of the stores fetches them again from the arguments and waits)
  int gm = g.M, gn = g.N;
  int64_t ldc = g.ldc;
  out_ptr cptr = (out_ptr)g.C;
  asm volatile("" : "+s"(gm), "+s"(gn), "+s"(ldc), "+s"(cptr));
  __syncthreads();                                   // every wave is done reading the stages
  if constexpr (F32OUT) {
    constexpr int CPW = 8 * T, PROWS = 64, RPI = 64 / CPW;      // chunks per row, rows of a patch (T / 2 in turn), rows per store
    static_assert(4 * PROWS * CPW * 8 <= NXS * XE + NWS * WE, "four patches");
    float* patch = (float*)smem + wave * (PROWS * CPW * 4);
    const int pp = lane % CPW, rsub = lane / CPW;
#pragma unroll
    for (int part = 0; part < T / 2; ++part) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int pr = 16 * i + l16;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          const f32x4_t& c = acc[4 * part + i][j];
          *(float4*)(patch + pr * (CPW * 4) + (((4 * j + gi) ^ (pr & (CPW - 1))) << 2)) = float4{c[0], c[1], c[2], c[3]};
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");        // the wave's own writes have landed; no other wave touches its patch
#pragma unroll
      for (int it = 0; it < PROWS / RPI; ++it) {
        const int pr = it * RPI + rsub;
        const out_u32x4 v = *(const out_u32x4*)(patch + pr * (CPW * 4) + pp * 4);
        const int m = m0 + wm + 64 * part + pr, n = n0 + wn + 4 * (pp ^ (pr & (CPW - 1)));
        if (m < gm && n < gn) __builtin_nontemporal_store(v, (out_u32x4_ptr)(cptr + ((int64_t)m * ldc + n) * 4));
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
  } else {
    constexpr int CPW = 4 * T;                       // chunks per patch row (32 T columns)
    constexpr int PROWS = 32 * T;                    // patch rows
    constexpr int RPI = 64 / CPW;                    // rows per store instruction
    static_assert(CPW <= 64 && 64 % CPW == 0 && PROWS % RPI == 0, "patch rows must tile a wave");
    static_assert(4 * PROWS * CPW * 8 <= NXS * XE + NWS * WE, "four patches");
    bf16_t* patch = smem + wave * (PROWS * CPW * 8);
    const int pp = lane % CPW, rsub = lane / CPW;
    if constexpr (RES) {
      // the residual's part of the tile lands in the wave's patch (zeros where a problem has none), where a lane finds its own
      // pieces and leaves the sums
      const __amdgpu_buffer_rsrc_t rrs = make_rsrc(g.R, g.R ? (int64_t)g.M * g.ldr * 2 : 0);
#pragma unroll
      for (int it = 0; it < PROWS / RPI; ++it) {
        const int pr = it * RPI + rsub;
        request16(rrs, patch + it * 512, (int)(((int64_t)(m0 + wm + pr) * g.ldr + n0 + wn + 8 * (pp ^ (pr & (CPW - 1)))) * 2));
      }
      __builtin_amdgcn_s_waitcnt(0x0F70);
      asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int pr = 16 * i + l16;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        uint2* at = (uint2*)(patch + pr * (CPW * 8) + (((2 * j + (gi >> 1)) ^ (pr & (CPW - 1))) << 3) + 4 * (gi & 1));
        // (here, not as soon as the wait is over: taken apart that early, accumulators were moved about and three were spilled)
        if constexpr (RES) asm volatile("" : "+a"(acc[i][j]));
        f32x4_t c = acc[i][j];
        if constexpr (RES) {
          const uint2 r = *at;
          c[0] += __uint_as_float(r.x << 16); c[1] += __uint_as_float(r.x & 0xffff0000u);
          c[2] += __uint_as_float(r.y << 16); c[3] += __uint_as_float(r.y & 0xffff0000u);
        }
        *at = uint2{pack_bf16x2(c[0], c[1]), pack_bf16x2(c[2], c[3])};
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the wave's own writes have landed; no other wave touches its patch
#pragma unroll
    for (int it = 0; it < PROWS / RPI; ++it) {
      const int pr = it * RPI + rsub;
      const out_u32x4 v = *(const out_u32x4*)(patch + pr * (CPW * 8) + pp * 8);
      const int m = m0 + wm + pr, n = n0 + wn + 8 * (pp ^ (pr & (CPW - 1)));
      if (m < gm && n < gn) __builtin_nontemporal_store(v, (out_u32x4_ptr)(cptr + ((int64_t)m * ldc + n) * 2));
    }
  }
}

// ---------------------------------------------------------------------------
// The same product for problems with too few 256 x 256 tiles for the chip: tiles of 128 WM x 128 WN, of which EVERY
// wave still accumulates 128 x 128 (256 accumulation registers), the KG = 4 / (WM WN) waves of one part of the tile
// taking the k steps of a slice between them.  What bounds a small tile is LDS bandwidth, not the matrix pipe: four
// waves of 64 x 64 read 32 fragments per 16 MFMAs, a wave of 128 x 128 reads 8, and the waves' sums meet once, in LDS,
// behind the loop.  Per slice of 64 k (128 x 128 tile, X k-contiguous, W row-contiguous, transpose reads at half rate): 768
// LDS cycles of reads + 256 of arriving data with four 64 x 64 waves, 384 + 256 this way, against 512 of MFMA.
// And a small tile's slice is over in some 700 cycles, less than a trip to memory: the slices go through a ring of NST
// LDS stages (five of 32 KB, or three of 48 KB), requested anew as soon as every wave has a slice's fragments, with explicit LDS
// reads and counted waits (the compiler would wait for every request before any LDS read).  Fragments of the next step are read
// behind the MFMAs of the current one; one barrier per slice.  Reads, requests and the cursors' scalar arithmetic each have
// their place behind an MFMA: in front of the barrier and behind it they cost 100 - 190 cycles per step.  Cycles per slice without
// loads / with loads that hit L2 / from memory, at 777 - 1531 rows of 4096 over 4096: 128 x 128 670 / 810 / 850 - 950 before, 560 /
// 640 / 690 - 840 now; 256 x 128 1400 / 1430 / 1420 - 1540 before, 1140 / 1090 / 1110 - 1370 now.
// ---------------------------------------------------------------------------
template <int WM, int WN, bool XK, bool WK, bool F32OUT>
__global__ __launch_bounds__(256, 1) void gemm_bf16_ksplit_kernel(GemmGroup grp) {
  constexpr int BM = 128 * WM, BN = 128 * WN;
  constexpr int KG = 4 / (WM * WN), KS = 4 / KG;    // waves per tile part; k steps of a slice per wave
  constexpr int XE = BM * BK, WE = BN * BK, SE = XE + WE;
  constexpr int NST = KG == 4 ? 5 : 3;
  __shared__ __attribute__((aligned(1024))) bf16_t smem[NST * SE];

  int pi, m0, n0;
  locate_tile<BM, BN>(grp, blockIdx.x, pi, m0, n0);
  const GemmArgs& g = grp.p[pi];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave % KG, wmn = wave / KG;
  const int wm = (WM == 2 ? wmn : 0) * 128, wn = (WN == 2 ? wmn : 0) * 128;

  // ---- request side
  constexpr int XLD = BM / 32, WLD = BN / 32, NLD = XLD + WLD;      // requests per thread and slice
  const int ldx = (int)g.lda, ldw = (int)g.ldb;
  int xoff[XLD], woff[WLD];
  auto chunk_off = [&](int q, bool kmajor, int rows, int ld) BEAGLE_INLINE_LAMBDA {                // 16-byte chunk q of an operand's slice
    if (kmajor) { const int r = q >> 3; return (r * ld + 8 * ((q & 7) ^ ((r >> 1) & 7))) * 2; }
    const int cpr = rows / 8, k = q / cpr;
    return (k * ld + 8 * ((q % cpr) ^ ((k & 3) << 2))) * 2;
  };
#pragma unroll
  for (int i = 0; i < XLD; ++i) xoff[i] = chunk_off(tid + 256 * i, XK, BM, ldx);
#pragma unroll
  for (int i = 0; i < WLD; ++i) woff[i] = chunk_off(tid + 256 * i, WK, BN, ldw);
  int nk = (g.K + BK - 1) / BK + (g.A2 ? (g.K2 + BK - 1) / BK : 0);
  SliceCursor fx, fw;
  fx.init(g, g.A, g.A2, XK, g.M, m0, ldx, BK, smem + wave * 512);
  fw.init(g, g.B, g.B2, WK, g.N, n0, ldw, BK, smem + XE + wave * 512);
  constexpr int PIECES = SliceCursor::PIECES;
  auto f_issue = [&](auto i_) BEAGLE_INLINE_LAMBDA {
    constexpr int i = decltype(i_)::value;
    if constexpr (i < XLD) request16(fx.rsrc, fx.dst + i * 2048, xoff[i]);
    else request16(fw.rsrc, fw.dst + (i - XLD) * 2048, woff[i - XLD]);
  };
  auto f_next = [&](auto i_) BEAGLE_INLINE_LAMBDA {
    constexpr int i = decltype(i_)::value;
    if constexpr (i < PIECES) fx.next<i, NST, SE>(); else fw.next<i - PIECES, NST, SE>();
  };

  // ---- fragment addresses (bytes) in the stage that is read next; everything else is an immediate
  typedef __attribute__((address_space(3))) bf16_t* lds_bf16_ptr;
  const uint32_t base = (uint32_t)(uintptr_t)(lds_bf16_ptr)smem;
  const int ql = lane & 31, hf = lane >> 5;
  // Accumulator row i of wave kg is row block (i + kg OWN) % 4 of its part: every wave then keeps its rows 0 .. OWN - 1 at
  // the exchange behind the loop, and no branch ever picks accumulators by wave.
  constexpr int OWN = 4 / KG;                        // 32-row blocks a wave keeps
  constexpr int NWA = WK ? KS : 4;
  uint32_t xa[XK ? KS : 1][4], wa[NWA];
  int xblk[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) xblk[i] = (i + kg * OWN) & 3;
  {
    const int gi = lane >> 4, r16 = lane & 15, kr = 8 * (gi >> 1) + (r16 >> 2);
    auto kmaj = [&](int r0, int s) BEAGLE_INLINE_LAMBDA { return ((r0 + ql) * BK + (((2 * (kg * KS + s) + hf) ^ ((ql >> 1) & 7)) << 3)) * 2; };
    auto rmaj = [&](int rows, int r0, int b) BEAGLE_INLINE_LAMBDA {
      const int col = r0 + 32 * b + 16 * (gi & 1) + 4 * (r16 & 3);
      return ((kg * KS * 16 + kr) * rows + ((((col >> 3) ^ ((kr & 3) << 2)) << 3) | (col & 7))) * 2;
    };
#pragma unroll
    for (int s = 0; s < (XK ? KS : 1); ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) xa[s][i] = base + (XK ? kmaj(wm + 32 * xblk[i], s) : rmaj(BM, wm, xblk[i]));
#pragma unroll
    for (int i = 0; i < NWA; ++i) wa[i] = base + 2 * XE + (WK ? kmaj(wn, i) : rmaj(BN, wn, i));
  }
  union frag_t { lds_u32x4_t u; struct { lds_u32x2_t a, b; } s; bf16x8_t v; };
  frag_t xf[2][4], wf[2][4];
  int r_st = 0, r_step = SE * 2;                     // the stage the addresses point into; bytes from there to the next
  auto r_next = [&]() BEAGLE_INLINE_LAMBDA { r_st = r_st + 1 == NST ? 0 : r_st + 1; r_step = r_st + 1 == NST ? -(NST - 1) * SE * 2 : SE * 2; };
  // LDS read n of step s of a slice: X fragments first (one read each, or two transpose reads), then W's; behind a slice's last read
  // of an address, it moves on to the next stage
  constexpr int NXR = XK ? 4 : 8, NWR = WK ? 4 : 8, NR = NXR + NWR;
  auto read_one = [&](auto fb_, auto s_, auto n_) BEAGLE_INLINE_LAMBDA {
    constexpr int fb = decltype(fb_)::value, s = decltype(s_)::value, n = decltype(n_)::value;
    if constexpr (n < NXR) {
      if constexpr (XK) lds_read_b128<0>(xf[fb][n].u, xa[s][n]);
      else if constexpr (n & 1) lds_read_tr16_b64<s * 16 * BM * 2 + 4 * BM * 2>(xf[fb][n >> 1].s.b, xa[0][n >> 1]);
      else lds_read_tr16_b64<s * 16 * BM * 2>(xf[fb][n >> 1].s.a, xa[0][n >> 1]);
      if constexpr (XK) xa[s][n] += r_step;
      else if constexpr (s == KS - 1 && (n & 1)) xa[0][n >> 1] += r_step;
    } else {
      constexpr int k = n - NXR;
      if constexpr (WK) lds_read_b128<k * 32 * BK * 2>(wf[fb][k].u, wa[s]);
      else if constexpr (k & 1) lds_read_tr16_b64<s * 16 * BN * 2 + 4 * BN * 2>(wf[fb][k >> 1].s.b, wa[k >> 1]);
      else lds_read_tr16_b64<s * 16 * BN * 2>(wf[fb][k >> 1].s.a, wa[k >> 1]);
      if constexpr (WK ? k == NWR - 1 : s == KS - 1 && (k & 1)) wa[WK ? s : k >> 1] += r_step;
    }
  };
  auto frags_wait = [&](auto fb_) BEAGLE_INLINE_LAMBDA {                  // the step's fragments are in registers; nothing that uses them moves up
    constexpr int fb = decltype(fb_)::value;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < 4; ++i) { lds_tie(xf[fb][i].u); lds_tie(wf[fb][i].u); }
  };

  f32x16_t acc[4][4];
  // f(j, q) for the 16 groups of four consecutive columns that a lane holds of a 32-row block
  auto quads = [&](auto f) BEAGLE_INLINE_LAMBDA {
    static_for<0, 16>([&](auto b_) BEAGLE_INLINE_LAMBDA { f(int_c<(decltype(b_)::value >> 2)>{}, int_c<(decltype(b_)::value & 3)>{}); });
  };
  // The requests of a slice go evenly over the MFMAs from a slice's last step to the next one's, but for the place of the cursors'
  // pieces behind them; FIRST of them fall in that last step.
  constexpr int SLOTS = 16 * KS, RS = KS == 1 ? SLOTS - 4 : SLOTS - 8, FIRST = KS == 1 ? NLD : 16 * NLD / RS;
  // the first slices, as far as a last step ahead of them would have come; the accumulators are cleared while they travel
  fx.describe(); fw.describe();
#pragma unroll 1
  for (int t = 0; t < NST - 1; ++t) { static_for<0, NLD>(f_issue); static_for<0, 2 * PIECES>(f_next); }
  static_for<0, FIRST>(f_issue);
  if constexpr (KS == 1) static_for<0, 2 * PIECES>(f_next);
  __builtin_amdgcn_sched_barrier(0);
  static_for<0, 16>([&](auto b_) BEAGLE_INLINE_LAMBDA {
    constexpr int b = decltype(b_)::value;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[b >> 2][b & 3][e] = 0.f;
  });
  __builtin_amdgcn_sched_barrier(0);

  auto landed = [&](auto n_) BEAGLE_INLINE_LAMBDA {                       // all but the n youngest requests have landed, for every wave
    constexpr int n = decltype(n_)::value;
    __builtin_amdgcn_s_waitcnt((n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // One slice; on entry its first step's fragments are in registers (parity P).  Before its last step the next slice has
  // landed for everybody and every wave has this slice's fragments in registers: its stage is requested anew, from that step to
  // the next slice's last.  Every MFMA is pinned in its place, with at most one or two reads, one request and one piece of the
  // cursors' arithmetic behind it.
  auto slice = [&](auto par_) BEAGLE_INLINE_LAMBDA {
    constexpr int P = decltype(par_)::value;
    static_for<0, KS>([&](auto s_) BEAGLE_INLINE_LAMBDA {
      constexpr int s = decltype(s_)::value, fb = (P + s) & 1;
      constexpr bool last = s + 1 == KS;
      constexpr int ns = last ? 0 : s + 1;
      if constexpr (last) landed(int_c<(NST - 2) * NLD>{});
      __builtin_amdgcn_sched_barrier(0);
      static_for<0, 16>([&](auto m_) BEAGLE_INLINE_LAMBDA {
        constexpr int m = decltype(m_)::value, i = m >> 2, j = (i & 1) ? 3 - (m & 3) : m & 3;
        mfma_in_place(acc[i][j], wf[fb][j].v, xf[fb][i].v);
        constexpr int r0 = m * NR * 5 / 64, r1 = (m + 1) * NR * 5 / 64;      // reads behind the first four fifths
        if constexpr (r0 < NR) static_for<r0, (r1 < NR ? r1 : NR)>([&](auto n_) BEAGLE_INLINE_LAMBDA { read_one(int_c<(fb ^ 1)>{}, int_c<ns>{}, n_); });
        constexpr int mm = last ? m : 16 + 16 * s + m;
        constexpr int d0 = mm * NLD / RS, d1 = (mm + 1) * NLD / RS;
        if constexpr (d0 < NLD) static_for<d0, (d1 < NLD ? d1 : NLD)>(f_issue);
        constexpr int pc = mm - RS, PP = KS == 1 ? 2 : 1;
        if constexpr (pc >= 0) { static_for<pc * PP, pc * PP + PP>(f_next); }
        if constexpr (s == 0 && m == 15) r_next();
        __builtin_amdgcn_sched_barrier(0);
      });
      frags_wait(int_c<(fb ^ 1)>{});
    });
  };
  static_assert(2 * PIECES == 8, "as many places behind the last request");

  landed(int_c<(NST - 2) * NLD + FIRST>{});          // slice 0
  static_for<0, NR>([&](auto n_) BEAGLE_INLINE_LAMBDA { read_one(int_c<0>{}, int_c<0>{}, n_); });
  if constexpr (KS == 1) r_next();
  frags_wait(int_c<0>{});
  int t = 0;
  if constexpr (KS % 2 == 0) {
#pragma unroll 1
    for (; t < nk; ++t) slice(int_c<0>{});
  } else {
#pragma unroll 1
    for (; t + 2 <= nk; t += 2) { slice(int_c<0>{}); slice(int_c<1>{}); }
    if (t < nk) slice(int_c<0>{});
  }
  mfma_drain();

  // ---- the KG waves of a tile part exchange sums: each ends up with 128 / KG of the rows, summed in a fixed order
  constexpr int SLOT = OWN * 4096;                   // floats of one wave's slot
  __builtin_amdgcn_s_waitcnt(0x0F70);                // the requests past the end (they write zeros) have landed
  __syncthreads();
  float* slot = nullptr;
  static_for<1, KG>([&](auto p_) BEAGLE_INLINE_LAMBDA {
    constexpr int p = decltype(p_)::value;           // rows p OWN .. go to the wave p further round, which keeps those blocks
    float* half = (float*)smem + (KG == 4 && (p & 1) == 0 ? 4 * SLOT : 0);
    float* out = half + (wmn * KG + (kg + p) % KG) * SLOT;
    static_for<0, OWN>([&](auto i_) BEAGLE_INLINE_LAMBDA {
      constexpr int i = decltype(i_)::value;
      quads([&](auto j_, auto q_) BEAGLE_INLINE_LAMBDA {
        constexpr int j = decltype(j_)::value, q = decltype(q_)::value;
        const f32x16_t& c = acc[p * OWN + i][j];
        *(float4*)(out + i * 4096 + ((4 * j + q) * 64 + lane) * 4) = float4{c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
      });
    });
    __syncthreads();
    slot = half + wave * SLOT;
    static_for<0, OWN>([&](auto i_) BEAGLE_INLINE_LAMBDA {
      constexpr int i = decltype(i_)::value;
      quads([&](auto j_, auto q_) BEAGLE_INLINE_LAMBDA {
        constexpr int j = decltype(j_)::value, q = decltype(q_)::value;
        const float4 v = *(const float4*)(slot + i * 4096 + ((4 * j + q) * 64 + lane) * 4);
        f32x16_t& c = acc[i][j];
        c[4 * q] += v.x; c[4 * q + 1] += v.y; c[4 * q + 2] += v.z; c[4 * q + 3] += v.w;
      });
    });
  });
  static_assert((KG == 4 ? 2 : 1) * 4 * SLOT * 4 <= NST * SE * 2, "the exchange must fit in the stages");

  // ---- rows out, through the wave's own slot of the last phase (nobody else touches it any more): whole row segments.
  // Chunk c (16 bytes) of patch row r sits at c ^ (r % chunks), which spreads the column-wise writes over the banks.
  // (the bounds in registers: otherwise every one of the stores fetches them again from the arguments and waits)
  int gm = g.M, gn = g.N;
  int64_t ldc = g.ldc;
  out_ptr cptr = (out_ptr)g.C;
  // Rows of a cache go past L2: the 64 KB of each of 256 tiles all leave at once.  Appends, us, no rows / V / K / both past L2: 1013 states
  // 71.7 / 70.2 / 70.7 / 69.6, 700 57.7 / 55.6 / 57.2 / 55.1, with K read back by its rotary embedding in the next launch; without one 1013
  // 66.9 / 65.5 / 65.2 / 64.6.  A training step's outputs do not: it cost 400 and 777 rows 0.5 %.
  const int kept = XK && !WK && !F32OUT ? g.c_kept : 0;
  asm volatile("" : "+s"(gm), "+s"(gn), "+s"(ldc), "+s"(cptr));
  static_for<0, OWN>([&](auto i_) BEAGLE_INLINE_LAMBDA {
    constexpr int i = decltype(i_)::value;
    const int mb = m0 + wm + 32 * (i + kg * OWN), nb = n0 + wn;
    if constexpr (F32OUT) {
      float* patch = slot + i * 4096;        // 32 rows x 128 floats: chunks of four, 32 per row
      quads([&](auto j_, auto q_) BEAGLE_INLINE_LAMBDA {
        constexpr int j = decltype(j_)::value, q = decltype(q_)::value;
        *(float4*)(patch + ql * 128 + (((8 * j + 2 * q + hf) ^ ql) << 2)) =
            float4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
      });
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int it = 0; it < 16; ++it) {
        const int r = 2 * it + hf, p = ql, m = mb + r, n = nb + 4 * (p ^ r);
        const out_u32x4 v = *(const out_u32x4*)(patch + r * 128 + 4 * p);
        if (m < gm && n < gn) *(out_u32x4_ptr)(cptr + ((int64_t)m * ldc + n) * 4) = v;
      }
    } else {
      bf16_t* patch = (bf16_t*)(slot + i * 4096);   // 32 rows x 128: 16 chunks of eight per row
      const int rr = lane >> 4, p = lane & 15;
      if (g.R) {                                     // residual: its rows in, the lanes' pieces out, added before the rounding
#pragma unroll
        for (int it = 0; it < 8; ++it) {
          const int r = 4 * it + rr, m = mb + r, n = nb + 8 * (p ^ (r & 15));
          uint4 v = {0, 0, 0, 0};
          if (m < gm && n < gn) v = *(const uint4*)((const bf16_t*)g.R + (int64_t)m * g.ldr + n);
          *(uint4*)(patch + r * 128 + 8 * p) = v;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        quads([&](auto j_, auto q_) BEAGLE_INLINE_LAMBDA {
          constexpr int j = decltype(j_)::value, q = decltype(q_)::value;
          const uint2 r = *(const uint2*)(patch + ql * 128 + (((4 * j + q) ^ (ql & 15)) << 3) + 4 * hf);
          acc[i][j][4 * q] += __uint_as_float(r.x << 16); acc[i][j][4 * q + 1] += __uint_as_float(r.x & 0xffff0000u);
          acc[i][j][4 * q + 2] += __uint_as_float(r.y << 16); acc[i][j][4 * q + 3] += __uint_as_float(r.y & 0xffff0000u);
        });
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
      quads([&](auto j_, auto q_) BEAGLE_INLINE_LAMBDA {
        constexpr int j = decltype(j_)::value, q = decltype(q_)::value;
        *(uint2*)(patch + ql * 128 + (((4 * j + q) ^ (ql & 15)) << 3) + 4 * hf) =
            uint2{pack_bf16x2(acc[i][j][4 * q], acc[i][j][4 * q + 1]), pack_bf16x2(acc[i][j][4 * q + 2], acc[i][j][4 * q + 3])};
      });
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      auto rows_out = [&](auto past_) BEAGLE_INLINE_LAMBDA {
#pragma unroll
        for (int it = 0; it < 8; ++it) {
          const int r = 4 * it + rr, m = mb + r, n = nb + 8 * (p ^ (r & 15));
          const out_u32x4 v = *(const out_u32x4*)(patch + r * 128 + 8 * p);
          const out_u32x4_ptr at = (out_u32x4_ptr)(cptr + ((int64_t)m * ldc + n) * 2);
          if (m < gm && n < gn) { if constexpr (decltype(past_)::value) __builtin_nontemporal_store(v, at); else *at = v; }
        }
      };
      if (kept) { rows_out(int_c<1>{}); asm volatile("; past L2" ::: "memory"); }      // (not the same code, or the compiler keeps one of the two)
      else rows_out(int_c<0>{});
    }
  });
}

// What the MFMA kernel needs of a group (checked by the entry points before anything is enqueued, see
// gemm_bf16_supported): k-contiguous operands with K a multiple of the k slice, every operand (and the residual)
// addressable through a 32-bit buffer descriptor, and one of the storage-order combinations instantiated below.
static bool group_fits(const GemmGroup& grp) {
  if (grp.count < 1 || grp.count > 4) return false;
  const bool xk = grp.p[0].a_kmajor, wk = grp.p[0].b_kmajor, f32 = grp.p[0].c_is_f32;
  const int64_t lim = (int64_t)1 << 31;
  bool res = false;
  for (int i = 0; i < grp.count; ++i) {
    const GemmArgs& q = grp.p[i];
    if ((bool)q.a_kmajor != xk || (bool)q.b_kmajor != wk || (bool)q.c_is_f32 != f32) return false;
    if (q.R) { res = true; if ((int64_t)q.M * q.ldr * 2 >= lim) return false; }
    if ((xk || wk) && (q.K % BK || (q.A2 && q.K2 % BK))) return false;
    if ((int64_t)(xk ? q.M : q.K) * q.lda * 2 >= lim || (int64_t)(wk ? q.N : q.K) * q.ldb * 2 >= lim) return false;
    if (q.A2 && (q.lda2 != q.lda || q.ldb2 != q.ldb)) return false;
    if (q.A2 && ((int64_t)(xk ? q.M : q.K2) * q.lda2 * 2 >= lim || (int64_t)(wk ? q.N : q.K2) * q.ldb2 * 2 >= lim)) return false;
  }
  if (res) return xk && !f32;
  return (xk && !f32) || (!xk && !wk);
}
bool gemm_bf16_supported(const GemmGroup& grp) { return group_fits(grp); }

static void check_group(const GemmGroup& grp) {
  if (!group_fits(grp)) {
    // The entry points refuse such problems with BEAGLE_ERR_UNSUPPORTED before they enqueue anything; there is no
    // slower kernel to fall back to.  Getting here is a bug in the library's own host code.
    fprintf(stderr, "beagle_xattn: internal error: GEMM group outside the MFMA kernel's domain reached the launcher\n");
    abort();
  }
}

template <int T>
static void launch_square(const GemmGroup& grp, hipStream_t s) {
  constexpr int BM = 64 * T;
  int total = 0;
  for (int i = 0; i < grp.count; ++i) total += ((grp.p[i].M + BM - 1) / BM) * ((grp.p[i].N + BM - 1) / BM);
  if (total == 0) return;
  const bool xk = grp.p[0].a_kmajor, wk = grp.p[0].b_kmajor, f32 = grp.p[0].c_is_f32;
  bool res = false;
  for (int i = 0; i < grp.count; ++i) if (grp.p[i].R) res = true;
  const dim3 grid(total), wg(256);
  if (res && !wk) hipLaunchKernelGGL((gemm_bf16_kernel<T, true, false, false, true>), grid, wg, 0, s, grp);
  else if (res) hipLaunchKernelGGL((gemm_bf16_kernel<T, true, true, false, true>), grid, wg, 0, s, grp);
  else if (xk && !wk) hipLaunchKernelGGL((gemm_bf16_kernel<T, true, false, false, false>), grid, wg, 0, s, grp);
  else if (xk) hipLaunchKernelGGL((gemm_bf16_kernel<T, true, true, false, false>), grid, wg, 0, s, grp);
  else if (!f32) hipLaunchKernelGGL((gemm_bf16_kernel<T, false, false, false, false>), grid, wg, 0, s, grp);
  else hipLaunchKernelGGL((gemm_bf16_kernel<T, false, false, true, false>), grid, wg, 0, s, grp);
}

template <int WM, int WN>
static void launch_ksplit(const GemmGroup& grp, hipStream_t s) {
  constexpr int BM = 128 * WM, BN = 128 * WN;
  int total = 0;
  for (int i = 0; i < grp.count; ++i)
    total += ((grp.p[i].M + BM - 1) / BM) * ((grp.p[i].N + BN - 1) / BN);
  if (total == 0) return;
  const bool xk = grp.p[0].a_kmajor, wk = grp.p[0].b_kmajor, f32 = grp.p[0].c_is_f32;
  const dim3 grid(total), wg(256);
  if (xk && !wk) hipLaunchKernelGGL((gemm_bf16_ksplit_kernel<WM, WN, true, false, false>), grid, wg, 0, s, grp);
  else if (xk) hipLaunchKernelGGL((gemm_bf16_ksplit_kernel<WM, WN, true, true, false>), grid, wg, 0, s, grp);
  else if (!f32) hipLaunchKernelGGL((gemm_bf16_ksplit_kernel<WM, WN, false, false, false>), grid, wg, 0, s, grp);
  else hipLaunchKernelGGL((gemm_bf16_ksplit_kernel<WM, WN, false, false, true>), grid, wg, 0, s, grp);
}

// Tile choice: what a launch takes with each tile size, from the number of tiles, the depth of each problem and how full
// the rounds (one workgroup per CU; two of the smallest kind) are.  A round costs a fixed part (first slices, exchange, stores) and
// so much per slice of 64 k, less when part of the chip is idle.  Fitted to 98 launches timed on their own (256 - 4096 rows of 4096
// over 256 - 11008, every storage order), to 6 - 10 % each; the choice is on average 0.6 % above the best tile's time, the worst
// 10 %.  Large problems come out at 256 x 256 by their operand traffic alone (1.45 PFLOP/s against 1.12 and 0.85).
// Tiles of 128 x 128 over a short contraction may take four waves of 64 x 64 instead (TILE_128_SHALLOW): no sums to exchange, half the
// accumulators to clear, and two workgroups per CU; but twice the LDS reads.  256 rows of 4096 over 256 / 1024 / 2048 / 4096, us:
// 11.9 / 15.6 / 21.0 / 31 with waves that split k, 8.5 / 13.2 / 19.7 / 37; 1024 over 2048 X^T Y 25.6, 25.7.
constexpr int SHALLOW = 16;                         // slices of 64 k
enum TileSize { TILE_256, TILE_256x128, TILE_128x256, TILE_128, TILE_128_SHALLOW };
struct TileChoice { TileSize tile; double us; };
struct TileCost { int bm, bn; double at_once, fixed, slice, slice_full; };

// Problems of different depth (dXkv contracts over two matrices, dXq over one): their tiles are dealt out in problem order,
// each to the place that is free first, so shallow tiles fill up behind deep ones, and a launch of less than a round lasts as long
// as its deepest tile.  By the mean depth 1024 positions at 5120 channels took 160 large tiles for their input gradients (whole
// backward 628 us, now 256 x 128 and 557), and the 320 tiles of 2500 positions were cut although their shallow half fills up the
// second round (866 -> 839); simulation step of 3048 positions 1386 -> 1351, 3 of 500 at 2048 channels 239 -> 226.
// `tiles` and `depth` of each of `count` problems; less than 0: too many rounds for the depths to matter.
static double uneven_us(const TileCost& c, const double* tiles, const double* depth, int count) {
  double total = 0.0;
  for (int i = 0; i < count; ++i) total += tiles[i];
  if (total > 4096.0) return -1.0;
  const double fill = total < c.at_once ? total / c.at_once : 1.0;
  struct { double at, cus; } free_at[64];            // CUs by the time they are free
  int n = 1;
  free_at[0] = {0.0, c.at_once};
  double end = 0.0;
  for (int i = 0; i < count; ++i) {
    const double us = c.fixed + depth[i] * (c.slice + c.slice_full * fill);
    for (double left = tiles[i]; left > 0.0;) {
      int e = 0;
      for (int k = 1; k < n; ++k) if (free_at[k].at < free_at[e].at) e = k;
      const double at = free_at[e].at + us, some = left < free_at[e].cus ? left : free_at[e].cus;
      left -= some;
      free_at[e].cus -= some;
      if (free_at[e].cus == 0.0) free_at[e] = free_at[--n];
      int k = 0;
      while (k < n && free_at[k].at != at) ++k;
      if (k == 64) return -1.0;
      if (k == n) free_at[n++] = {at, some}; else free_at[k].cus += some;
      if (at > end) end = at;
    }
  }
  return end;
}

static TileChoice choose_tile(const GemmGroup& grp) {
  static const TileCost costs[] = {{256, 256, 256.0, 7.0, 0.91, 0.46}, {256, 128, 256.0, 6.7, 0.45, 0.38}, {128, 256, 256.0, 6.7, 0.45, 0.38},
                                   {128, 128, 256.0, 5.9, 0.29, 0.21}, {128, 128, 512.0, 2.7, 0.285, 0.66}};      // by TileSize
  int best = 0;
  double best_us = 0.0;
  for (int c = 0; c < 5; ++c) {
    double tiles = 0.0, slices = 0.0;               // slices: over all tiles
    double each[4], deep[4];                        // tiles and depth of each problem
    bool even = true;
    for (int i = 0; i < grp.count; ++i) {
      const GemmArgs& q = grp.p[i];
      const double t = (double)((q.M + costs[c].bm - 1) / costs[c].bm) * ((q.N + costs[c].bn - 1) / costs[c].bn);
      each[i] = t;
      deep[i] = (q.K + BK - 1) / BK + (q.A2 ? (q.K2 + BK - 1) / BK : 0);
      even = even && deep[i] == deep[0];
      tiles += t;
      slices += t * deep[i];
    }
    if (tiles == 0.0) continue;
    const double depth = slices / tiles, full = floor(tiles / costs[c].at_once), rest = tiles / costs[c].at_once - full;
    if (c == TILE_128_SHALLOW && depth > SHALLOW) continue;
    double us = full * (costs[c].fixed + depth * (costs[c].slice + costs[c].slice_full));
    if (rest > 0.0) us += costs[c].fixed + depth * (costs[c].slice + costs[c].slice_full * rest);
    if (!even) {
      const double uneven = uneven_us(costs[c], each, deep, grp.count);
      if (uneven >= 0.0) us = uneven;
    }
    if (c == 0 || us < best_us) { best = c; best_us = us; }
  }
  return {(TileSize)best, best_us};
}

static void launch_chosen(const GemmGroup& grp, TileSize tile, hipStream_t s) {
  switch (tile) {
    case TILE_256: return launch_square<4>(grp, s);
    case TILE_256x128: return launch_ksplit<2, 1>(grp, s);
    case TILE_128x256: return launch_ksplit<1, 2>(grp, s);
    case TILE_128: return launch_ksplit<1, 1>(grp, s);
    case TILE_128_SHALLOW: return launch_square<2>(grp, s);
  }
}

// A few 256 x 256 tiles past a whole number of rounds hold the chip for most of another round (3048 x 11008 x 4096: 516 tiles,
// by the costs above 66 us for the last four after two rounds of 108).  The bottom tile rows of one problem that make up the
// excess then go into a launch of their own, on small tiles that spread them over the chip (37 us).  The same costs decide,
// with CUT_US for the second launch and for what the fit is off.  Whole calls, us: training step of 4100 positions, 32 heads
// 2134 -> 2057, of 4224 in 8 groups 1835 -> 1790, of 3400 at 5120 channels 2535 -> 2503; draft block on 3048 packed rows
// 4341 -> 4277.  Past half a round of excess the costs find nothing (7.5 rounds of 8192 positions at 5120 channels stay whole).
constexpr double CUT_US = 8.0;
static bool cut_excess(const GemmGroup& grp, double whole_us, GemmGroup* main, GemmGroup* rest) {
  int tiles = 0;
  for (int i = 0; i < grp.count; ++i) tiles += ((grp.p[i].M + 255) / 256) * ((grp.p[i].N + 255) / 256);
  const int excess = tiles % 256;
  if (tiles < 256 || excess == 0 || excess > 128) return false;
  double best_us = whole_us - CUT_US;
  bool found = false;
  for (int i = 0; i < grp.count; ++i) {
    const GemmArgs& q = grp.p[i];
    const int rows = (q.M + 255) / 256, cols = (q.N + 255) / 256, r = (excess + cols - 1) / cols;
    // a row-contiguous X read from the middle of its rows: only whole tiles stay inside the matrix in its last k row
    if (r >= rows || (!q.a_kmajor && q.M % 256)) continue;
    GemmGroup a = grp, b; memset(&b, 0, sizeof(b));
    const int64_t m0 = (int64_t)(rows - r) * 256;
    a.p[i].M = (int32_t)m0;
    b.count = 1;
    GemmArgs& t = b.p[0];
    t = q;
    t.M = (int32_t)(q.M - m0);
    t.A = (const bf16_t*)q.A + m0 * (q.a_kmajor ? q.lda : 1);
    if (q.A2) t.A2 = (const bf16_t*)q.A2 + m0 * (q.a_kmajor ? q.lda2 : 1);
    t.C = (char*)q.C + m0 * q.ldc * (q.c_is_f32 ? 4 : 2);
    if (q.R) t.R = (const bf16_t*)q.R + m0 * q.ldr;
    const double us = choose_tile(a).us + choose_tile(b).us;
    if (us < best_us) { best_us = us; *main = a; *rest = b; found = true; }
  }
  return found;
}

// Every GEMM of a group must share storage orders and output type; the hot
// path only forms such groups.  Supported: X k-major with W either order
// (forward projections, input gradients), both row-major-in-k (weight grads).
void launch_gemm_bf16(const GemmGroup& grp, hipStream_t s, const char* name) {
  ProfScope ps(name, s);
  check_group(grp);
  const TileChoice whole = choose_tile(grp);
  GemmGroup main, rest;
  if (whole.tile == TILE_256 && cut_excess(grp, whole.us, &main, &rest)) {
    launch_chosen(main, choose_tile(main).tile, s);
    launch_chosen(rest, choose_tile(rest).tile, s);
    return;
  }
  launch_chosen(grp, whole.tile, s);
}

template <bool F32OUT>
__global__ __launch_bounds__(256) void sum_pairs_kernel(SumPairArgs p, int64_t n4) {
  const int t = blockIdx.y;
  const float4* a = (const float4*)p.a[t];
  const float4* b = (const float4*)p.b[t];
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256) {
    const float4 x = a[i], y = b[i];
    const float4 v = {x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w};
    if (F32OUT) ((float4*)p.out[t])[i] = v;
    else ((uint2*)p.out[t])[i] = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
  }
}
void launch_sum_pairs(const SumPairArgs& p, int64_t n, bool out_f32, hipStream_t s, const char* name) {
  ProfScope ps(name, s);
  const int64_t n4 = n / 4;
  const dim3 grid((unsigned)((n4 + 255) / 256 < 2048 ? (n4 + 255) / 256 : 2048), p.count);
  if (out_f32) hipLaunchKernelGGL(sum_pairs_kernel<true>, grid, dim3(256), 0, s, p, n4);
  else hipLaunchKernelGGL(sum_pairs_kernel<false>, grid, dim3(256), 0, s, p, n4);
}

}  // namespace beagle
