// bf16 GEMM on the gfx950 matrix cores: C[M,N] = X * W (+ X2 * W2), float
// accumulation, for the Q/K/V/output projections of Eq. 2 and every
// projection-shaped contraction of the backward pass.
//
// Design
//   * One workgroup of 4 wavefronts (2 x 2) owns a 256 x 256 tile of C (128 x
//     128 for a few shallow products); each wave owns a quarter of it as T x T
//     accumulators of the v_mfma_f32_32x32x16_bf16 instruction.
//   * The k loop walks BK = 64 at a time through two LDS stages.  Slices go
//     from HBM/L2 straight into LDS (buffer_load ... lds, 16 bytes per lane):
//     no staging registers, no ds_write, and out-of-range chunks arrive as
//     zeros through the buffer descriptor's range check.  The loads of slice
//     t+1 are issued before the MFMAs of slice t; one vmcnt wait + barrier per
//     slice.  The two stages are two separate __shared__ arrays so that the
//     compiler can tell a fragment read of one stage from an in-flight load
//     into the other.
//   * Each operand tile sits in LDS in the order it has in HBM (a lane's 16
//     bytes land at wave_base + 16 * lane), with an XOR swizzle chosen on the
//     GLOBAL side (which chunk a lane fetches) so that reads are conflict free:
//       k-contiguous operand  -> rows of 128 B; chunk c of row r is stored at
//                                chunk c ^ ((r >> 1) & 7); a fragment is one
//                                ds_read_b128;
//       row-contiguous operand-> k-rows of ROWS*2 B; chunk c of k-row k is
//                                stored at chunk c ^ ((k & 3) << 2); a fragment
//                                is two ds_read_b64_tr_b16 (the LDS transpose
//                                read), which hand every lane four consecutive
//                                k of its own row.
//   * Fragments are double-buffered in registers: those of k step s+1 are read
//     from LDS before the MFMAs of step s are issued.
//   * The MFMA is issued "transposed" (A operand = W rows, B operand = X rows)
//     so that a lane ends up with 4 consecutive n of one C row in 4 consecutive
//     accumulator registers: the epilogue stores 8 (bf16) or 16 (float) bytes
//     per lane per instruction.
//   * Workgroup ids are remapped so that each XCD (ids are dealt round-robin
//     to the 8 XCDs) works on a contiguous run of tiles, and tiles are walked
//     in groups of GROUP_M tile-rows so that the run shares X and W tiles in
//     that XCD's L2.
//   * Several independent GEMMs can share one launch (Q, K, V projections;
//     the three weight gradients) so that small ones do not leave CUs idle.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include "common.h"

namespace beagle {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4_t;
typedef s16x4_t __attribute__((address_space(3))) * lds_s16x4_ptr;
typedef __attribute__((address_space(3))) void* lds_void_ptr;

constexpr int BK = 64;
constexpr int GROUP_M = 4;
constexpr int NUM_XCD = 8;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)bytes, 0x00020000);
}

// 16 bytes per lane, HBM/L2 -> LDS at dst + 16 * lane
__device__ __forceinline__ void request16(__amdgpu_buffer_rsrc_t rsrc, bf16_t* dst, int off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)dst, 16, off, 0, 0, 0);
}

// One BK slice of one operand, HBM -> LDS.  Chunk q = tid + 256 i of the tile
// (16 bytes) lands at tile + 16 q; which global chunk it is follows from the
// swizzle.
//   KMAJOR : element (row r, k) at base[r * ld + k]   (buffer = rows * ld elements)
//   !KMAJOR: element (row r, k) at base[k * ld + r]   (buffer = K * ld elements)
// k beyond K must read as zero: for !KMAJOR that is past the end of the buffer;
// for KMAJOR the launcher requires K % BK == 0.  Rows beyond the matrix only
// feed output rows/columns that are never stored, so whatever they read (zero
// past the end, or a neighbouring row) is harmless.
template <int ROWS, bool KMAJOR>
__device__ __forceinline__ void load_slice(bf16_t* tile, __amdgpu_buffer_rsrc_t rsrc, int64_t ld, int row0, int k0,
                                           int tid) {
  constexpr int PER_THREAD = ROWS * BK / 8 / 256;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
  for (int i = 0; i < PER_THREAD; ++i) {
    const int q = tid + 256 * i;
    int off;
    if (KMAJOR) {
      const int r = q >> 3, c = (q & 7) ^ ((r >> 1) & 7);
      off = (int)(((int64_t)(row0 + r) * ld + k0 + 8 * c) * 2);
    } else {
      constexpr int CPR = ROWS / 8;
      const int k = q / CPR, c = (q % CPR) ^ ((k & 3) << 2);
      off = (int)(((int64_t)(k0 + k) * ld + row0 + 8 * c) * 2);
    }
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(tile + (i * 4 + wave) * 512), 16, off, 0, 0, 0);
  }
}

// Per-lane element offsets of an operand's fragments inside its tile, computed
// once per kernel.  Everything that varies inside the k loop (the 32-row block
// for k-contiguous tiles, the k step for both) is then a compile-time constant
// added to one of these, i.e. an immediate offset of the LDS read.
//   KMAJOR : o[ks]  = row (l % 32), swizzled chunk of k step ks       (+ 32-row block * BK)
//   !KMAJOR: o[blk] = k-row (8 (l/32) + (l%16)/4), swizzled column of block blk   (+ k step * 16 * ROWS)
template <int ROWS, bool KMAJOR, int NBLK>
struct FragOffs {
  int o[KMAJOR ? BK / 16 : NBLK];
  __device__ __forceinline__ void init(int lane, int r0) {
    if (KMAJOR) {
      const int ql = lane & 31, hf = lane >> 5;
#pragma unroll
      for (int ks = 0; ks < BK / 16; ++ks) o[ks] = (r0 + ql) * BK + (((2 * ks + hf) ^ ((ql >> 1) & 7)) << 3);
    } else {
      const int gi = lane >> 4, r16 = lane & 15;
      const int kr = 8 * (gi >> 1) + (r16 >> 2);
#pragma unroll
      for (int b = 0; b < NBLK; ++b) {
        const int col = r0 + 32 * b + 16 * (gi & 1) + 4 * (r16 & 3);
        o[b] = kr * ROWS + ((((col >> 3) ^ ((kr & 3) << 2)) << 3) | (col & 7));
      }
    }
  }
};

// MFMA operand fragment: lane l gets row (r0 + 32 blk + l % 32), k = 16 ks + 8 * (l / 32) .. + 7.
template <int ROWS, bool KMAJOR, int NBLK>
__device__ __forceinline__ bf16x8_t read_frag(const bf16_t* tile, const FragOffs<ROWS, KMAJOR, NBLK>& f, int blk, int ks) {
  if (KMAJOR) {
    return *(const bf16x8_t*)(tile + blk * 32 * BK + f.o[ks]);
  } else {
    // transpose read: the 16 lanes of a group pass the addresses of 4 k-rows x
    // 4 pieces of 4 rows; lane l of the group receives k-rows 0..3 of row l.
    const bf16_t* p = tile + ks * 16 * ROWS + f.o[blk];
    union { struct { s16x4_t a, b; } s; bf16x8_t v; } u;
    u.s.a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)p);
    u.s.b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * ROWS));
    return u.v;
  }
}

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
  constexpr int TM = T, TN = T;                  // 32 x 32 accumulators per wave
  constexpr int BM = 64 * TM, BN = 64 * TN;
  constexpr int XE = BM * BK, WE = BN * BK;      // elements per operand tile
  __shared__ __attribute__((aligned(1024))) bf16_t stage0[XE + WE];
  __shared__ __attribute__((aligned(1024))) bf16_t stage1[XE + WE];

  int pi, m0, n0;
  locate_tile<BM, BN>(grp, blockIdx.x, pi, m0, n0);
  const GemmArgs& g = grp.p[pi];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave >> 1) * (32 * TM), wn = (wave & 1) * (32 * TN);

  FragOffs<BM, XK, TM> xo;
  FragOffs<BN, WK, TN> wo;
  xo.init(lane, wm);
  wo.init(lane, wn);

  // The accumulators are cleared behind the first segment's first requests, not ahead of them: 256 register
  // writes per lane are 2 000 cycles that the first round trip to memory can hide.
  f32x16_t acc[TM][TN];
  auto clear_acc = [&]() {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  };
  bool fresh = true;

#pragma unroll 1
  for (int seg = 0; seg < 2; ++seg) {
    const bf16_t* X = (const bf16_t*)(seg ? g.A2 : g.A);
    const bf16_t* W = (const bf16_t*)(seg ? g.B2 : g.B);
    const int K = seg ? g.K2 : g.K;
    const int64_t ldx = seg ? g.lda2 : g.lda, ldw = seg ? g.ldb2 : g.ldb;
    if (X == nullptr || K <= 0) continue;
    const int nk = (K + BK - 1) / BK;
    const __amdgpu_buffer_rsrc_t xrs = make_rsrc(X, (int64_t)(XK ? g.M : K) * ldx * 2);
    const __amdgpu_buffer_rsrc_t wrs = make_rsrc(W, (int64_t)(WK ? g.N : K) * ldw * 2);

    bf16x8_t xf[2][TM], wf[2][TN];
    auto fetch_x = [&](bf16_t* st, int k0) { load_slice<BM, XK>(st, xrs, ldx, m0, k0, tid); };
    auto fetch_w = [&](bf16_t* st, int k0) { load_slice<BN, WK>(st + XE, wrs, ldw, n0, k0, tid); };
    auto frags = [&](const bf16_t* st, int fb, int ks) {
#pragma unroll
      for (int i = 0; i < TM; ++i) xf[fb][i] = read_frag<BM, XK, TM>(st, xo, i, ks);
#pragma unroll
      for (int j = 0; j < TN; ++j) wf[fb][j] = read_frag<BN, WK, TN>(st + XE, wo, j, ks);
    };
    auto mfmas = [&](int fb) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[fb][j], xf[fb][i], acc[i][j], 0, 0, 0);
    };
    constexpr int NSTEP = BK / 16;                                      // k steps per slice (4)
    constexpr int NREADS = (XK ? TM : 2 * TM) + (WK ? TN : 2 * TN);     // LDS reads per k step
    constexpr int XLOADS = BM * BK / 8 / 256, WLOADS = BN * BK / 8 / 256;   // HBM->LDS loads per thread per slice
    static_assert(NSTEP == 4 && NREADS % 2 == 0 && NREADS / 2 <= TM * TN, "issue pattern below assumes this");
    static_assert(XLOADS <= TM * TN && WLOADS <= TM * TN, "one load per MFMA at most");
    // One k slice.  On entry: slice kt is visible in `cur` and its step-0 fragments are in
    // registers; the X half of slice kt+1 is already on its way into `nxt`.
    //   step 0    : MFMAs + LDS reads of step 1 + the W half of slice kt+1 (one load per MFMA)
    //   steps 1,2 : MFMAs + LDS reads of the next step
    //   wait for this thread's loads, barrier: slice kt+1 visible, nobody reads `cur` any more
    //   step 3    : MFMAs from registers + first fragment reads of slice kt+1 + the X half of
    //               slice kt+2 into `cur`
    // so every HBM->LDS load is issued at least two k steps (>= 1000 cycles) before it is
    // waited for, and the in-order wave never waits on a queue while the MFMA pipe is idle.
    auto slice = [&](bf16_t* cur, bf16_t* nxt, int kt) {
      fetch_w(nxt, (kt + 1) * BK);    // past the last slice these fetch zeros / unused rows: harmless
#pragma unroll
      for (int ks = 0; ks < NSTEP - 1; ++ks) {
        const int fb = ks & 1;
        frags(cur, fb ^ 1, ks + 1);
        mfmas(fb);
#pragma unroll
        for (int t = 0; t < TM * TN; ++t) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if (t < NREADS / 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
          if (ks == 0 && t < WLOADS) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        }
      }
      __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this thread's chunks of the next slice are in LDS
      __syncthreads();                      // everyone's are, and everyone is done reading `cur`
      frags(nxt, 0, 0);
      fetch_x(cur, (kt + 2) * BK);
      mfmas((NSTEP - 1) & 1);
#pragma unroll
      for (int t = 0; t < TM * TN; ++t) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (t < NREADS / 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        if (t < XLOADS) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
    };

    __syncthreads();                        // previous segment: all reads done, both stages free
    fetch_x(stage0, 0);
    fetch_w(stage0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (fresh) { clear_acc(); fresh = false; }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    frags(stage0, 0, 0);
    fetch_x(stage1, BK);
    int kt = 0;
#pragma unroll 1
    for (; kt + 2 <= nk; kt += 2) {
      slice(stage0, stage1, kt);
      slice(stage1, stage0, kt + 1);
    }
    if (kt < nk) slice(stage0, stage1, kt);
    __builtin_amdgcn_s_waitcnt(0x0F70);     // drain the look-ahead loads before the stages are reused
  }
  if (fresh) clear_acc();                   // no segment at all: C = 0 (+ residual)

  // ---- residual operand: its tile goes HBM -> LDS in one burst (both stages are free now), so that the
  // epilogue below does not pay one HBM round trip per store.  Chunk q = tid + 256 i (16 bytes) of the tile
  // lands at 16 q; chunk position pc of row r holds global chunk pc ^ (r % CPR), which spreads the epilogue's
  // same-column reads of 32 different rows over the banks.  The upper half of the rows lives in stage1.
  constexpr int CPR = BN / 8;                      // 16-byte chunks per tile row
  constexpr int RLOADS = BM * CPR / 256;           // per thread
  const bool with_res = RES && !F32OUT && g.R != nullptr;
  if (with_res) {
    static_assert((BM / 2) * BN <= XE + WE, "half of the residual tile must fit one stage");
    __syncthreads();                               // every wave is done reading the operand stages
    const __amdgpu_buffer_rsrc_t rrs = make_rsrc(g.R, (int64_t)g.M * g.ldr * 2);
#pragma unroll
    for (int i = 0; i < RLOADS; ++i) {
      const int q = tid + 256 * i, r = q / CPR, c = (q % CPR) ^ (r & (CPR - 1));
      const int off = (int)(((int64_t)(m0 + r) * g.ldr + n0 + 8 * c) * 2);
      bf16_t* st = i < RLOADS / 2 ? stage0 : stage1;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rrs, (lds_void_ptr)(st + ((i % (RLOADS / 2)) * 4 + wave) * 512), 16, off,
                                               0, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
  }

  // ---- epilogue: lane holds C row m = .. + lane % 32; register e of tile (i, j)
  // holds column n = .. + 8 * (e / 4) + 4 * (lane / 32) + e % 4.
  if constexpr (F32OUT) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = m0 + wm + 32 * i + (lane & 31);
      if (m >= g.M) continue;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int n = n0 + wn + 32 * j + 8 * q + 4 * (lane >> 5);
          if (n >= g.N) continue;
          float4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          *(float4*)((float*)g.C + (int64_t)m * g.ldc + n) = v;
        }
      }
    }
  } else {
    // bf16 output.  Straight from the registers a store instruction would carry 16 bytes for each of 32 rows, and
    // the workgroup -- the only one on its CU -- spent 15 % of its life issuing them (measured: 27 500 cycles per
    // 256 x 256 tile against 2 350 per k slice).  Each wave therefore transposes its part of the tile through a
    // patch of LDS of its own (the operand stages are free now; two patches per stage) and writes whole row
    // segments: 16 bytes per lane, 64 / CPW rows per instruction.  Patch rows hold CPW 16-byte chunks; chunk c
    // of row r sits at position c ^ (r % CPW), which spreads the column-wise writes over the banks.
    constexpr int CPW = 4 * TN;                      // chunks per patch row (32 TN columns)
    constexpr int PROWS = 32 * TM;                   // patch rows
    constexpr int RPI = 64 / CPW;                    // rows per store instruction
    static_assert(CPW <= 64 && 64 % CPW == 0 && PROWS % RPI == 0, "patch rows must tile a wave");
    static_assert(2 * PROWS * CPW * 8 <= XE + WE, "two patches per stage");
    if (with_res) {
      // the residual tile occupies the stages: take it into the accumulators first, then let go of it
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int rt = wm + 32 * i + (lane & 31);      // row inside the tile
        const bf16_t* rrow = (rt < BM / 2 ? stage0 : stage1) + (rt % (BM / 2)) * BN;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int ct = wn + 32 * j + 8 * q;        // first column of this 8-column chunk inside the tile
            const uint2 r = *(const uint2*)(rrow + (((ct >> 3) ^ (rt & (CPR - 1))) << 3) + 4 * (lane >> 5));
            acc[i][j][4 * q] += __uint_as_float(r.x << 16); acc[i][j][4 * q + 1] += __uint_as_float(r.x & 0xffff0000u);
            acc[i][j][4 * q + 2] += __uint_as_float(r.y << 16); acc[i][j][4 * q + 3] += __uint_as_float(r.y & 0xffff0000u);
          }
      }
    }
    __syncthreads();                                 // every wave is done reading the stages
    bf16_t* patch = (wave < 2 ? stage0 : stage1) + (wave & 1) * (PROWS * CPW * 8);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int pr = 32 * i + (lane & 31);
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          uint2 v = {pack_bf16x2(acc[i][j][4 * q], acc[i][j][4 * q + 1]), pack_bf16x2(acc[i][j][4 * q + 2], acc[i][j][4 * q + 3])};
          *(uint2*)(patch + pr * (CPW * 8) + (((4 * j + q) ^ (pr & (CPW - 1))) << 3) + 4 * (lane >> 5)) = v;
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the wave's own writes have landed; no other wave touches its patch
    const int pp = lane % CPW, rsub = lane / CPW;
    // (the bounds in registers: otherwise every one of the 32 stores fetches them again from the arguments and waits)
    int gm = g.M, gn = g.N;
    asm volatile("" : "+s"(gm), "+s"(gn));
#pragma unroll
    for (int it = 0; it < PROWS / RPI; ++it) {
      const int pr = it * RPI + rsub;
      const uint4 v = *(const uint4*)(patch + pr * (CPW * 8) + pp * 8);
      const int m = m0 + wm + pr, n = n0 + wn + 8 * (pp ^ (pr & (CPW - 1)));
      if (m < gm && n < gn) { typedef unsigned int nt_u32x4 __attribute__((ext_vector_type(4))); const nt_u32x4 w = {v.x, v.y, v.z, v.w}; __builtin_nontemporal_store(w, (nt_u32x4*)((bf16_t*)g.C + (int64_t)m * g.ldc + n)); }
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
// LDS stages (four of 32 KB, or three of 48 KB), requested NST slices ahead, with explicit LDS reads and counted
// waits (the compiler would wait for every request before any LDS read).  Fragments of the next step are read behind
// the MFMAs of the current one; one barrier per slice.
// ---------------------------------------------------------------------------
template <int WM, int WN, bool XK, bool WK, bool F32OUT>
__global__ __launch_bounds__(256, 1) void gemm_bf16_ksplit_kernel(GemmGroup grp) {
  constexpr int BM = 128 * WM, BN = 128 * WN;
  constexpr int KG = 4 / (WM * WN), KS = 4 / KG;    // waves per tile part; k steps of a slice per wave
  constexpr int XE = BM * BK, WE = BN * BK, SE = XE + WE;
  constexpr int NST = SE * 2 * 4 <= 128 * 1024 ? 4 : 3;
  __shared__ __attribute__((aligned(1024))) bf16_t smem[NST * SE];

  int pi, m0, n0;
  locate_tile<BM, BN>(grp, blockIdx.x, pi, m0, n0);
  const GemmArgs& g = grp.p[pi];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave % KG, wmn = wave / KG;
  const int wm = (WM == 2 ? wmn : 0) * 128, wn = (WN == 2 ? wmn : 0) * 128;

  // ---- request side: a cursor over the slices of both k segments.  The descriptors start at the current slice, so the
  // lanes' offsets are constants of the tile and a slice costs scalar arithmetic only; past the last slice they are empty.
  const int nk1 = (g.K + BK - 1) / BK, nk = nk1 + (g.A2 ? (g.K2 + BK - 1) / BK : 0);
  constexpr int XLD = BM / 32, WLD = BN / 32;        // requests per thread and slice
  const int ldx = (int)g.lda, ldw = (int)g.ldb;
  int xoff[XLD], woff[WLD];
#pragma unroll
  for (int i = 0; i < XLD; ++i) {
    const int q = tid + 256 * i;
    if (XK) { const int r = q >> 3; xoff[i] = (r * ldx + 8 * ((q & 7) ^ ((r >> 1) & 7))) * 2; }
    else { constexpr int CPR = BM / 8; const int k = q / CPR; xoff[i] = (k * ldx + 8 * ((q % CPR) ^ ((k & 3) << 2))) * 2; }
  }
#pragma unroll
  for (int i = 0; i < WLD; ++i) {
    const int q = tid + 256 * i;
    if (WK) { const int r = q >> 3; woff[i] = (r * ldw + 8 * ((q & 7) ^ ((r >> 1) & 7))) * 2; }
    else { constexpr int CPR = BN / 8; const int k = q / CPR; woff[i] = (k * ldw + 8 * ((q % CPR) ^ ((k & 3) << 2))) * 2; }
  }
  const char *fx, *fw;                               // current slice of this tile's rows
  int64_t xleft, wleft;                              // bytes from there to the operand's end
  auto seek = [&](const void* X, const void* W, int K) BEAGLE_INLINE_LAMBDA {
    const int64_t xo = XK ? (int64_t)m0 * ldx * 2 : (int64_t)m0 * 2, wo = WK ? (int64_t)n0 * ldw * 2 : (int64_t)n0 * 2;
    fx = (const char*)X + xo; xleft = (int64_t)(XK ? g.M : K) * ldx * 2 - xo;
    fw = (const char*)W + wo; wleft = (int64_t)(WK ? g.N : K) * ldw * 2 - wo;
  };
  seek(g.A, g.B, g.K);
  const int64_t xstep = XK ? BK * 2 : (int64_t)BK * ldx * 2, wstep = WK ? BK * 2 : (int64_t)BK * ldw * 2;
  int f_t = 0, f_st = 0;                             // next slice to request, its stage
  __amdgpu_buffer_rsrc_t xrs, wrs;
  bf16_t* f_dst;
  auto f_begin = [&]() BEAGLE_INLINE_LAMBDA {
    if (f_t == nk1 && f_t < nk) seek(g.A2, g.B2, g.K2);
    xrs = make_rsrc(fx, f_t < nk && xleft > 0 ? xleft : 0);
    wrs = make_rsrc(fw, f_t < nk && wleft > 0 ? wleft : 0);
    f_dst = smem + f_st * SE + wave * 512;
    fx += xstep; xleft -= xstep; fw += wstep; wleft -= wstep;
    ++f_t; f_st = f_st + 1 == NST ? 0 : f_st + 1;
  };
  auto f_issue = [&](auto i_) BEAGLE_INLINE_LAMBDA {
    constexpr int i = decltype(i_)::value;
    if constexpr (i < XLD) request16(xrs, f_dst + i * 2048, xoff[i]);
    else request16(wrs, f_dst + XE + (i - XLD) * 2048, woff[i - XLD]);
  };
  constexpr int NLD = XLD + WLD;

  // ---- fragment addresses (bytes from the start of a stage); everything else is an immediate
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
  // LDS read n of a step: X fragments first (one read each, or two transpose reads), then W's
  constexpr int NXR = XK ? 4 : 8, NWR = WK ? 4 : 8;
  auto read_one = [&](auto fb_, auto s_, auto n_, uint32_t st) BEAGLE_INLINE_LAMBDA {
    constexpr int fb = decltype(fb_)::value, s = decltype(s_)::value, n = decltype(n_)::value;
    if constexpr (n < NXR) {
      if constexpr (XK) lds_read_b128<0>(xf[fb][n].u, xa[s][n] + st);
      else if constexpr (n & 1) lds_read_tr16_b64<s * 16 * BM * 2 + 4 * BM * 2>(xf[fb][n >> 1].s.b, xa[0][n >> 1] + st);
      else lds_read_tr16_b64<s * 16 * BM * 2>(xf[fb][n >> 1].s.a, xa[0][n >> 1] + st);
    } else {
      constexpr int k = n - NXR;
      if constexpr (WK) lds_read_b128<k * 32 * BK * 2>(wf[fb][k].u, wa[s] + st);
      else if constexpr (k & 1) lds_read_tr16_b64<s * 16 * BN * 2 + 4 * BN * 2>(wf[fb][k >> 1].s.b, wa[k >> 1] + st);
      else lds_read_tr16_b64<s * 16 * BN * 2>(wf[fb][k >> 1].s.a, wa[k >> 1] + st);
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
  // the first NST slices; the accumulators are cleared while they travel
#pragma unroll 1
  for (int t = 0; t < NST; ++t) { f_begin(); static_for<0, NLD>(f_issue); }
  __builtin_amdgcn_sched_barrier(0);
  static_for<0, 16>([&](auto b_) BEAGLE_INLINE_LAMBDA {
    constexpr int b = decltype(b_)::value;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[b >> 2][b & 3][e] = 0.f;
  });
  __builtin_amdgcn_sched_barrier(0);

  auto wait_slice = [&]() BEAGLE_INLINE_LAMBDA {                          // all but the NST - 2 youngest slices have landed, for every wave
    constexpr int n = (NST - 2) * NLD;
    __builtin_amdgcn_s_waitcnt((n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  uint32_t rst = 0;                                  // stage of the slice being read, in bytes
  // One slice; on entry its first step's fragments are in registers (parity P).  In its last step the next slice has
  // landed for everybody, every wave has this slice's fragments in registers, and this slice's stage is requested anew.
  auto slice = [&](auto par_) BEAGLE_INLINE_LAMBDA {
    constexpr int P = decltype(par_)::value;
    static_for<0, KS>([&](auto s_) BEAGLE_INLINE_LAMBDA {
      constexpr int s = decltype(s_)::value, fb = (P + s) & 1;
      constexpr bool last = s + 1 == KS;
      constexpr int ns = last ? 0 : s + 1;
      if constexpr (last) {
        wait_slice();
        f_begin();
        rst = rst + 2 * SE == NST * 2 * SE ? 0 : rst + 2 * SE;
      }
      const uint32_t st = rst;
      __builtin_amdgcn_sched_barrier(0);
      static_for<0, 16>([&](auto m_) BEAGLE_INLINE_LAMBDA {
        constexpr int m = decltype(m_)::value, i = m >> 2, j = m & 3;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[fb][j].v, xf[fb][i].v, acc[i][j], 0, 0, 0);
        // the next step's reads behind the first eight MFMAs, the requests behind the last ones
        constexpr int r0 = m * (NXR + NWR) / 8, r1 = (m + 1) * (NXR + NWR) / 8;
        if constexpr (m < 8) static_for<r0, r1>([&](auto n_) BEAGLE_INLINE_LAMBDA { read_one(int_c<(fb ^ 1)>{}, int_c<ns>{}, n_, st); });
        // one request every KS * 16 / NLD MFMAs, from the barrier on: a wave gets rid of a request in about a hundred
        // cycles, and issued faster than that it only stands in front of the MFMAs behind it
        constexpr int mm = last ? m : 16 + 16 * s + m;
        constexpr int d0 = (mm * NLD + 16 * KS - 1) / (16 * KS), d1 = ((mm + 1) * NLD + 16 * KS - 1) / (16 * KS);
        if constexpr (d1 > d0) f_issue(int_c<d0>{});
        __builtin_amdgcn_sched_barrier(0);
      });
      frags_wait(int_c<(fb ^ 1)>{});
    });
  };
  static_assert(NLD <= 16, "at most one request per MFMA");

  {
    constexpr int n = (NST - 1) * NLD;               // slice 0
    __builtin_amdgcn_s_waitcnt((n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    static_for<0, NXR + NWR>([&](auto n_) BEAGLE_INLINE_LAMBDA { read_one(int_c<0>{}, int_c<0>{}, n_, 0u); });
    frags_wait(int_c<0>{});
  }
  int t = 0;
  if constexpr (KS % 2 == 0) {
#pragma unroll 1
    for (; t < nk; ++t) slice(int_c<0>{});
  } else {
#pragma unroll 1
    for (; t + 2 <= nk; t += 2) { slice(int_c<0>{}); slice(int_c<1>{}); }
    if (t < nk) slice(int_c<0>{});
  }

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
        const float4 v = *(const float4*)(patch + r * 128 + 4 * p);
        if (m < g.M && n < g.N) *(float4*)((float*)g.C + (int64_t)m * g.ldc + n) = v;
      }
    } else {
      bf16_t* patch = (bf16_t*)(slot + i * 4096);   // 32 rows x 128: 16 chunks of eight per row
      const int rr = lane >> 4, p = lane & 15;
      if (g.R) {                                     // residual: its rows in, the lanes' pieces out, added before the rounding
#pragma unroll
        for (int it = 0; it < 8; ++it) {
          const int r = 4 * it + rr, m = mb + r, n = nb + 8 * (p ^ (r & 15));
          uint4 v = {0, 0, 0, 0};
          if (m < g.M && n < g.N) v = *(const uint4*)((const bf16_t*)g.R + (int64_t)m * g.ldr + n);
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
#pragma unroll
      for (int it = 0; it < 8; ++it) {
        const int r = 4 * it + rr, m = mb + r, n = nb + 8 * (p ^ (r & 15));
        const uint4 v = *(const uint4*)(patch + r * 128 + 8 * p);
        if (m < g.M && n < g.N) *(uint4*)((bf16_t*)g.C + (int64_t)m * g.ldc + n) = v;
      }
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
// the rounds of 256 workgroups (one per CU) are.  A round costs a fixed part (first slices, exchange, stores) and so much
// per slice of 64 k, less when part of the chip is idle.  Fitted to launches timed on their own, microseconds:
//   256 x 256: K 777 full 28; K 4096 full 107-122, a quarter full 76; K 11008 three quarters full 243
//   256 x 128, 128 x 256: K 777 full 20; K 4096 full 64-70, half full 52
//   128 x 128: K 777 full 13; K 4096 full 40, 7/8 full 36 (four waves of 64 x 64 per tile took 59)
// Large problems come out at 256 x 256 by their operand traffic alone (1.30 PFLOP/s against 0.95 and 0.80).
// Tiles of 128 x 128 over a short contraction take four waves of 64 x 64 instead (TILE_128_SHALLOW): no ring to fill and no sums
// to exchange, and half the accumulators to clear.  Two products of 768 x 1024 over K 128 / 512 / 1024, us: 10.2 / 12.6 / 15.8 with waves
// that split k -> 5.9 / 8.7 / 12.3; at K 1536 both take 19.3, at 2048 22.7 -> 24.5.
constexpr int SHALLOW = 16;                         // slices of 64 k
enum TileSize { TILE_256, TILE_256x128, TILE_128x256, TILE_128, TILE_128_SHALLOW };
struct TileChoice { TileSize tile; double us; };
struct TileCost { int bm, bn; double fixed, slice, slice_full; };

// Problems of different depth (dXkv contracts over two matrices, dXq over one): their tiles are dealt out in problem order,
// each to the CU that is free first, so shallow tiles fill up behind deep ones, and a launch of less than a round lasts as long
// as its deepest tile.  By the mean depth 1024 positions at 5120 channels took 160 large tiles for their input gradients (whole
// backward 628 us, now 256 x 128 and 557), and the 320 tiles of 2500 positions were cut although their shallow half fills up the
// second round (866 -> 839); simulation step of 3048 positions 1386 -> 1351, 3 of 500 at 2048 channels 239 -> 226.
// `tiles` and `depth` of each of `count` problems; less than 0: too many rounds for the depths to matter.
static double uneven_us(const TileCost& c, const double* tiles, const double* depth, int count) {
  double total = 0.0;
  for (int i = 0; i < count; ++i) total += tiles[i];
  if (total > 4096.0) return -1.0;
  const double fill = total < 256.0 ? total / 256.0 : 1.0;
  struct { double at, cus; } free_at[64];            // CUs by the time they are free
  int n = 1;
  free_at[0] = {0.0, 256.0};
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
  static const TileCost costs[] = {{256, 256, 8.8, 0.90, 0.65}, {256, 128, 8.3, 0.57, 0.38}, {128, 256, 8.3, 0.57, 0.38}, {128, 128, 6.1, 0.38, 0.16}};
  int best = 0;
  double best_us = 0.0, best_depth = 0.0;
  for (int c = 0; c < 4; ++c) {
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
    const double depth = slices / tiles, full = floor(tiles / 256.0), rest = tiles / 256.0 - full;
    double us = full * (costs[c].fixed + depth * (costs[c].slice + costs[c].slice_full));
    if (rest > 0.0) us += costs[c].fixed + depth * (costs[c].slice + costs[c].slice_full * rest);
    if (!even) {
      const double uneven = uneven_us(costs[c], each, deep, grp.count);
      if (uneven >= 0.0) us = uneven;
    }
    if (c == 0 || us < best_us) { best = c; best_us = us; best_depth = depth; }
  }
  if (best == TILE_128 && best_depth <= SHALLOW) best = TILE_128_SHALLOW;
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
