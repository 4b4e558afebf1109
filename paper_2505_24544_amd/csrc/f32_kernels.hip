// The fp32 path (io_dtype == BEAGLE_F32): projections and masked attention (attn_f32.h) in
// float throughout, on the float matrix instruction v_mfma_f32_16x16x4_f32 (an
// ordinary float multiply-add chain: results stay within 1e-5 of float64).
//
// The problems this path sees are small (the reference problem is 128 rows of
// 256), so what bounds it is latency: launches, trips to memory and serial
// chains, not arithmetic.  Hence:
//   * No LDS staging.  Operand fragments go from L2 straight into registers in
//     the matrix instruction's layout, 16 bytes at a time: the two operands only
//     have to agree on what k a lane group stands for, and which of a tile's columns
//     is an instruction's n-th is free.
//   * Small tiles (16 x 64 and half of that, 16 x 16 scores) whose eight waves split the
//     contraction, so that a 128 x 256 output occupies 64 workgroups and a
//     contraction of 256 is one trip to memory and 16 instructions of 32 cycles per
//     wave; the eight sums meet in LDS.  (Wide models' tiles: 32 x 64.)
//   * Everything independent shares a launch: problems of different storage
//     orders in one GEMM group, dQ with dK / dV in one attention launch.
// One training step at 128 rows, hidden 256, 4 heads of 64: 367 us on scalar
// kernels (nine launches), 46.5 on 32 x 32 x 2 instructions and four waves, 34.7 now.
#include <string.h>
#include "attn_f32.h"
#include "f32_plan.h"

namespace beagle {
namespace {

// A group and where each of its problems' tiles begin.  A workgroup finds its problem in one trip to the kernel's arguments and has all
// that the problem says in a second one (walking from problem to problem took a trip each).
struct TiledGroup {
  int32_t first[6];                                                    // from the launch's first tile on; past the last problem: beyond every tile
  GemmArgs p[6];
};
__device__ __forceinline__ const GemmArgs& problem_of(const TiledGroup& grp, int& t) {
  asm volatile("" :: "s"(grp.first[0]), "s"(grp.first[1]), "s"(grp.first[2]), "s"(grp.first[3]), "s"(grp.first[4]), "s"(grp.first[5]));
  int pi = 0, f = grp.first[0];
#pragma unroll
  for (int i = 1; i < 6; ++i)
    if (t >= grp.first[i]) { pi = i; f = grp.first[i]; }
  t -= f;
  const GemmArgs& p = grp.p[pi];
  asm volatile("" :: "s"(p.A), "s"(p.B), "s"(p.C), "s"(p.M), "s"(p.N), "s"(p.K), "s"(p.lda), "s"(p.ldb), "s"(p.ldc), "s"(p.a_kmajor),
               "s"(p.b_kmajor), "s"(p.A2), "s"(p.B2), "s"(p.K2), "s"(p.lda2), "s"(p.ldb2), "s"(p.R), "s"(p.ldr));
  return p;
}

// ---------------------------------------------------------------------------
// GEMM: a tile of 16 MR x 16 NU per workgroup, whose eight waves take chunks of 32 k in turn; the eight sums meet in LDS.
// Bound by one trip to memory and the chain behind it.  Lane (n, g) of a 16 x 16 x 4 instruction supplies row (column) n at k = g, and
// what it stands for is free: k = 16 j + 4 g + e of a chunk, so that a k-contiguous operand comes 16 bytes at a time, and column
// 4 n + u of the tile in instruction u, so that a row-contiguous B does too (10 requests per 32 k, and 32 instructions of 32 cycles;
// 32 x 32 tiles on 32 x 32 x 2 instructions took 20 requests, 16 of them of 4 bytes, and with four waves twice the chain).
// Every N and leading dimension is a multiple of 4, and so is K where an operand is k-contiguous (the descriptor's checks on widths).
// AHEAD: two chunks of a wave in flight, which leaves registers for one workgroup per CU; without, several share one.
// MR = 2: B's fragments serve two blocks of rows (12 requests for 64 instructions): wide problems, which tiles of 16 rows make a
// stream of B out of L2, take two thirds of the time.  Launches at hidden 4096, us, MR = 1 / 2: 2048 rows through Wo 993 / 727, the
// input and weight gradients behind them 3250 / 2320.  NU = 2: tiles of 32 columns, twice as many workgroups for a few rows.
// (Measured and not taken: 64 x 64 whose waves share the contraction four ways, 5 - 7 % faster than 32 x 64 at 1000 rows of 5120, 70 % slower
// at 128 of 4096; 32 x 64 a chunk ahead, 3 - 10 % slower.  f32_plan.h says which tiles a launch takes.)
// ---------------------------------------------------------------------------
constexpr int GW = 8;
template <int MR, int NU, bool AHEAD, bool ALONE>
__global__ __launch_bounds__(64 * GW, ALONE || MR > 1 ? 2 : 4) void gemm_f32_kernel(TiledGroup grp) {
  constexpr int GM = 16 * MR, GN = 16 * NU;
  typedef float bvec_t __attribute__((ext_vector_type(NU)));
  typedef float ovec_t __attribute__((ext_vector_type(NU / 2)));
  // (more than half of the CU's LDS: nothing else fits, and the compiler spends the registers)
  constexpr int SUMS = ALONE ? 81920 / (GM * (GN + 4) * 4) + 1 : GW;
  __shared__ __attribute__((aligned(16))) float red[SUMS][GM][GN + 4];
  int t = blockIdx.x;
  const GemmArgs& p = problem_of(grp, t);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, nl = lane & 15;
  const int tn = (p.N + GN - 1) / GN, m0 = (t / tn) * GM, n0 = (t % tn) * GN;
  const int nc = min(n0 + NU * nl, p.N - NU);                              // rows and columns past the end repeat the last ones
  int mr[MR];
  f32x4_t acc[MR][NU];
#pragma unroll
  for (int i = 0; i < MR; ++i) {
    mr[i] = min(m0 + 16 * i + nl, p.M - 1);
#pragma unroll
    for (int u = 0; u < NU; ++u) acc[i][u] = zero4();
  }

  // AK / BK: k contiguous in memory
  auto contract = [&](auto ak_, auto bk_) BEAGLE_INLINE_LAMBDA {
    constexpr bool AK = decltype(ak_)::value, BK = decltype(bk_)::value;
    // chunk c of both segments' 32 k each: register 4 j + e is k = 16 j + 4 g + e of it; past K: zeros on both sides (0 * inf is a NaN)
    const int nc1 = (p.K + 31) / 32, chunks = nc1 + (p.A2 ? (p.K2 + 31) / 32 : 0);
    auto load = [&](int c, float (&a)[MR][8], float (&b)[NU][8]) BEAGLE_INLINE_LAMBDA {
      const bool two = c >= nc1;
      const float* A = (const float*)(two ? p.A2 : p.A);
      const float* B = (const float*)(two ? p.B2 : p.B);
      const int64_t lda = two ? p.lda2 : p.lda, ldb = two ? p.ldb2 : p.ldb;
      const int K = two ? p.K2 : p.K, k0 = 32 * (two ? c - nc1 : c);
      auto at = [&](int k, int i, bool in) BEAGLE_INLINE_LAMBDA {      // one k of the operands that are not k-contiguous
        if (!AK) {
#pragma unroll
          for (int r = 0; r < MR; ++r) { const float v = A[k * lda + mr[r]]; a[r][i] = in ? v : 0.f; }
        }
        if (!BK) {
          const bvec_t v = *(const bvec_t*)(B + k * ldb + nc);
#pragma unroll
          for (int u = 0; u < NU; ++u) b[u][i] = in ? v[u] : 0.f;
        }
      };
      auto four = [&](int k, int j, bool in) BEAGLE_INLINE_LAMBDA {    // four of those that are
        auto put = [&](float (&f)[8], const float4& v) BEAGLE_INLINE_LAMBDA {
          f[4 * j] = in ? v.x : 0.f; f[4 * j + 1] = in ? v.y : 0.f; f[4 * j + 2] = in ? v.z : 0.f; f[4 * j + 3] = in ? v.w : 0.f;
        };
        if (AK) {
#pragma unroll
          for (int r = 0; r < MR; ++r) put(a[r], *(const float4*)(A + mr[r] * lda + k));
        }
        if (BK) {
#pragma unroll
          for (int u = 0; u < NU; ++u) put(b[u], *(const float4*)(B + (nc + u) * ldb + k));
        }
      };
      if (k0 + 32 <= K) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int k = k0 + 16 * j + 4 * g;
          four(k, j, true);
#pragma unroll
          for (int e = 0; e < 4; ++e) at(k + e, 4 * j + e, true);
        }
      } else {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int k = k0 + 16 * j + 4 * g;
          if (AK || BK) four(min(k, K - 4), j, k < K);
#pragma unroll
          for (int e = 0; e < 4; ++e) at(min(k + e, K - 1), 4 * j + e, k + e < K);
        }
      }
    };
    auto compute = [&](const float (&a)[MR][8], const float (&b)[NU][8]) BEAGLE_INLINE_LAMBDA {
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
          for (int r = 0; r < MR; ++r) acc[r][u] = mfma16(a[r][i], b[u][i], acc[r][u]);
    };
    // (AHEAD: a contraction of up to 512 is loaded whole before the first product)
    float a0[MR][8], b0[NU][8], a1[MR][8], b1[NU][8];
    int c = wave;
    if constexpr (!AHEAD) {
      for (; c < chunks; c += GW) {
        load(c, a0, b0);
        if constexpr (ALONE) {                                         // (piece by piece, as they land, wide launches took 3 - 8 % longer)
          __builtin_amdgcn_s_waitcnt(0x0F70);                          // vmcnt(0)
          __builtin_amdgcn_sched_barrier(0);
        }
        compute(a0, b0);
      }
      return;
    }
    if (c < chunks) load(c, a0, b0);
    if (c + GW < chunks) load(c + GW, a1, b1);
    for (; c < chunks; c += 2 * GW) {
      compute(a0, b0);
      if (c + 2 * GW < chunks) load(c + 2 * GW, a0, b0);
      if (c + GW < chunks) {
        compute(a1, b1);
        if (c + 3 * GW < chunks) load(c + 3 * GW, a1, b1);
      }
    }
  };
  if (p.a_kmajor && p.b_kmajor) contract(int_c<1>{}, int_c<1>{});
  else if (p.a_kmajor) contract(int_c<1>{}, int_c<0>{});
  else contract(int_c<0>{}, int_c<0>{});

#pragma unroll
  for (int i = 0; i < MR; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      bvec_t v;
#pragma unroll
      for (int u = 0; u < NU; ++u) v[u] = acc[i][u][e];
      *(bvec_t*)&red[wave][16 * i + 4 * g + e][NU * nl] = v;
    }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < MR; ++i) {                     // 32 threads to a row
    const int r = 16 * i + (tid >> 5), c = NU / 2 * (tid & 31), m = m0 + r, n = n0 + c;
    if (m >= p.M || n >= p.N) return;
    ovec_t v = *(const ovec_t*)&red[0][r][c];
#pragma unroll
    for (int w = 1; w < GW; ++w) v += *(const ovec_t*)&red[w][r][c];
    if (p.R) v += *(const ovec_t*)((const float*)p.R + m * p.ldr + n);
    *(ovec_t*)((float*)p.C + m * p.ldc + n) = v;
  }
}

}  // namespace

void launch_gemm_f32(const GemmGroup& g, hipStream_t s, const char* name) {
  F32Problem sh[6];
  for (int i = 0; i < g.count; ++i) sh[i] = {g.p[i].M, g.p[i].N, (g.p[i].K + 31) / 32 + (g.p[i].A2 ? (g.p[i].K2 + 31) / 32 : 0)};
  const F32Plan plan = gemm_f32_plan(sh, g.count);
  if (plan.tiles == 0) return;
  int64_t first[6], tiles = 0;
  for (int i = 0; i < g.count; ++i) { first[i] = tiles; tiles += gemm_f32_tiles(sh[i], plan.rows, plan.cols); }
  TiledGroup t;
  memcpy(t.p, g.p, sizeof(t.p));
  ProfScope ps(name, s);
  for_launches(tiles, 64 * GW, [&](int64_t at, int64_t n) {            // (2^31 tiles and more would not fit the memory)
    for (int i = 0; i < 6; ++i) t.first[i] = i < g.count ? (int32_t)(first[i] - at) : INT32_MAX;
    const dim3 grid((unsigned)n), wg(64 * GW);
    if (plan.rows == 32 && plan.alone) hipLaunchKernelGGL((gemm_f32_kernel<2, 4, false, true>), grid, wg, 0, s, t);
    else if (plan.rows == 32) hipLaunchKernelGGL((gemm_f32_kernel<2, 4, false, false>), grid, wg, 0, s, t);
    else if (plan.cols == 32) hipLaunchKernelGGL((gemm_f32_kernel<1, 2, false, false>), grid, wg, 0, s, t);
    else if (plan.ahead) hipLaunchKernelGGL((gemm_f32_kernel<1, 4, true, true>), grid, wg, 0, s, t);
    else hipLaunchKernelGGL((gemm_f32_kernel<1, 4, false, false>), grid, wg, 0, s, t);
  });
}

// the instantiation of a head width: 32-channel blocks, and whether they are full
template <class F>
static void launch_widths(const AttnArgs& a, F&& go) {
  auto full = [&](auto nc_) { if (a.d == 32 * decltype(nc_)::value) go(nc_, int_c<1>{}); else go(nc_, int_c<0>{}); };
  if (a.d <= 32) full(int_c<1>{}); else if (a.d <= 64) full(int_c<2>{}); else if (a.d <= 96) full(int_c<3>{}); else full(int_c<4>{});
}

void launch_attn_fwd_f32(const AttnArgs& a, hipStream_t s) {
  ProfScope ps("attn_fwd_f32", s);
  const int nq = (a.S + AT - 1) / AT;
  launch_widths(a, [&](auto nc_, auto full_) {
    for_launches(nq, 64 * AW, [&](int64_t at, int64_t n) {
      hipLaunchKernelGGL((attn_fwd_f32_kernel<decltype(nc_)::value, decltype(full_)::value>), dim3((unsigned)n, a.H, a.B), dim3(64 * AW), 0, s, a,
                         nq - 1 - (int)at);
    });
  });
}

void launch_attn_bwd_f32(const AttnArgs& a, hipStream_t s) {
  ProfScope ps("attn_bwd_f32", s);
  const int64_t nq = (a.S + AT - 1) / AT, nk = (a.L + AT - 1) / AT, rows_q = (int64_t)a.H * a.B, rows_kv = (int64_t)a.G * a.B;
  launch_widths(a, [&](auto nc_, auto full_) {
    for_launches(rows_q * nq + rows_kv * nk, 64 * AW, [&](int64_t at, int64_t n) {
      hipLaunchKernelGGL((attn_bwd_f32_kernel<decltype(nc_)::value, decltype(full_)::value>), dim3((unsigned)n), dim3(64 * AW), 0, s, a,
                         grid_part(at, n, rows_q, nq, nk));
    });
  });
}

}  // namespace beagle
