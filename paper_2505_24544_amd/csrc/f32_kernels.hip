// The fp32 path (io_dtype == BEAGLE_F32): projections and masked attention (attn_f32.h) in
// float throughout, on the float matrix instruction v_mfma_f32_32x32x2_f32 (an
// ordinary float multiply-add chain: results stay within 1e-5 of float64).
//
// The problems this path sees are small (the reference problem is 128 rows of
// 256), so what bounds it is latency: launches, trips to memory and serial
// chains, not arithmetic.  Hence:
//   * No LDS staging.  Operand fragments go from L2 straight into registers in
//     the matrix instruction's layout: lane l supplies row (column) l % 32, and
//     since the two operands only have to agree on what k a lane half stands
//     for, half h takes k = 8 i + 4 h + e of instruction (i, e): one 16-byte load
//     where k is contiguous in memory, four coalesced 4-byte loads where it is not.
//   * Small tiles (32 x 32) whose four waves split the contraction, so that a
//     128 x 256 output still occupies 32 workgroups and a contraction of 256 is
//     one trip to memory and 32 instructions per wave; the four sums meet in LDS.
//   * Everything independent shares a launch: problems of different storage
//     orders in one GEMM group, dQ with dK / dV in one attention launch.
// One training step at 128 rows, hidden 256, 4 heads of 64: 367 us with the
// scalar kernels that were here (nine launches of 27 - 87 us), 48 us now.
#include "attn_f32.h"

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
// GEMM.  KG = 4: a 32 x 32 tile per workgroup, the four waves take chunks of 32 k in turn.  KG = 1: a 64 x 64 tile, a
// 32 x 32 quarter per wave, for problems with tiles enough (half the operand traffic per flop).
// ---------------------------------------------------------------------------
template <int KG>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmGroup grp) {
  constexpr int T = KG == 4 ? 32 : 64;
  __shared__ float red[KG == 4 ? 4 : 1][32][33];
  int t = blockIdx.x, pi = 0;
  for (; pi + 1 < grp.count; ++pi) {
    const int n = ((grp.p[pi].M + T - 1) / T) * ((grp.p[pi].N + T - 1) / T);
    if (t < n) break;
    t -= n;
  }
  const GemmArgs& g = grp.p[pi];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), hf = lane >> 5, ql = lane & 31;
  const int tn = (g.N + T - 1) / T;
  const int m0 = (t / tn) * T + (KG == 1 ? (wave >> 1) * 32 : 0), n0 = (t % tn) * T + (KG == 1 ? (wave & 1) * 32 : 0);
  const int mr = min(m0 + ql, g.M - 1), nc = min(n0 + ql, g.N - 1);    // rows and columns past the end repeat the last one
  f32x16_t acc = zero16();

  // one k segment; AK / BK: k contiguous in memory
  auto segment = [&](auto ak_, auto bk_, const float* A, const float* B, int K, int64_t lda, int64_t ldb) BEAGLE_INLINE_LAMBDA {
    constexpr bool AK = decltype(ak_)::value, BK = decltype(bk_)::value;
    const float* ap = AK ? A + mr * lda : A + mr;
    const float* bp = BK ? B + nc * ldb : B + nc;
    // 32 k of both operands: register 4 i + e is k = k0 + 8 i + 4 hf + e; past K: zeros on both sides (0 * inf is a NaN)
    auto load = [&](int k0, float (&a)[16], float (&b)[16]) BEAGLE_INLINE_LAMBDA {
      if (k0 + 32 <= K) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int k = k0 + 8 * i + 4 * hf;
          if (AK) { const float4 v = *(const float4*)(ap + k); a[4 * i] = v.x; a[4 * i + 1] = v.y; a[4 * i + 2] = v.z; a[4 * i + 3] = v.w; }
          if (BK) { const float4 v = *(const float4*)(bp + k); b[4 * i] = v.x; b[4 * i + 1] = v.y; b[4 * i + 2] = v.z; b[4 * i + 3] = v.w; }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (!AK) a[4 * i + e] = ap[(k + e) * lda];
            if (!BK) b[4 * i + e] = bp[(k + e) * ldb];
          }
        }
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int k = k0 + 8 * (i >> 2) + 4 * hf + (i & 3), kc = min(k, K - 1);
          const float v = AK ? ap[kc] : ap[kc * lda], w = BK ? bp[kc] : bp[kc * ldb];
          a[i] = k < K ? v : 0.f;
          b[i] = k < K ? w : 0.f;
        }
      }
    };
    auto compute = [&](const float (&a)[16], const float (&b)[16]) BEAGLE_INLINE_LAMBDA {
#pragma unroll
      for (int i = 0; i < 16; ++i) acc = mfma(a[i], b[i], acc);
    };
    // two chunks in flight; a contraction of up to 256 (64 with one wave) is loaded whole before the first product
    float a0[16], b0[16], a1[16], b1[16];
    int k = KG == 4 ? 32 * wave : 0;
    constexpr int STEP = 32 * KG;
    if (k < K) load(k, a0, b0);
    if (k + STEP < K) load(k + STEP, a1, b1);
    for (; k < K; k += 2 * STEP) {
      compute(a0, b0);
      if (k + 2 * STEP < K) load(k + 2 * STEP, a0, b0);
      if (k + STEP < K) {
        compute(a1, b1);
        if (k + 3 * STEP < K) load(k + 3 * STEP, a1, b1);
      }
    }
  };
  auto both = [&](auto ak_, auto bk_) BEAGLE_INLINE_LAMBDA {
    segment(ak_, bk_, (const float*)g.A, (const float*)g.B, g.K, g.lda, g.ldb);
    if (g.A2) segment(ak_, bk_, (const float*)g.A2, (const float*)g.B2, g.K2, g.lda2, g.ldb2);
  };
  if (g.a_kmajor && g.b_kmajor) both(int_c<1>{}, int_c<1>{});
  else if (g.a_kmajor) both(int_c<1>{}, int_c<0>{});
  else both(int_c<0>{}, int_c<0>{});

  float* C = (float*)g.C;
  const float* R = (const float*)g.R;
  if (KG == 4) {
#pragma unroll
    for (int e = 0; e < 16; ++e) red[wave][acc_row(e, hf)][ql] = acc[e];
    __syncthreads();
    const int r = tid >> 3, c = (tid & 7) * 4, m = m0 + r;
    if (m < g.M) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int n = n0 + c + u;
        if (n >= g.N) break;
        float v = ((red[0][r][c + u] + red[KG == 4 ? 1 : 0][r][c + u]) + red[KG == 4 ? 2 : 0][r][c + u]) + red[KG == 4 ? 3 : 0][r][c + u];
        if (R) v += R[m * g.ldr + n];
        C[m * g.ldc + n] = v;
      }
    }
  } else {
    const int n = n0 + ql;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int m = m0 + acc_row(e, hf);
      if (m < g.M && n < g.N) C[m * g.ldc + n] = acc[e] + (R ? R[m * g.ldr + n] : 0.f);
    }
  }
}

}  // namespace

// 32 x 32 tiles while they are fewer than fit the chip twice over at four workgroups per CU; 64 x 64 beyond
void launch_gemm_f32(const GemmGroup& g, hipStream_t s, const char* name) {
  int64_t t32 = 0, t64 = 0;
  for (int i = 0; i < g.count; ++i) {
    t32 += (int64_t)((g.p[i].M + 31) / 32) * ((g.p[i].N + 31) / 32);
    t64 += (int64_t)((g.p[i].M + 63) / 64) * ((g.p[i].N + 63) / 64);
  }
  if (t32 == 0) return;
  ProfScope ps(name, s);
  if (t32 < 2048) hipLaunchKernelGGL(gemm_f32_kernel<4>, dim3((unsigned)t32), dim3(256), 0, s, g);
  else hipLaunchKernelGGL(gemm_f32_kernel<1>, dim3((unsigned)t64), dim3(256), 0, s, g);
}

// the instantiation of a head width: 32-channel blocks, and whether they are full
template <class F>
static void launch_widths(const AttnArgs& a, F&& go) {
  auto full = [&](auto nc_) { if (a.d == 32 * decltype(nc_)::value) go(nc_, int_c<1>{}); else go(nc_, int_c<0>{}); };
  if (a.d <= 32) full(int_c<1>{}); else if (a.d <= 64) full(int_c<2>{}); else if (a.d <= 96) full(int_c<3>{}); else full(int_c<4>{});
}

void launch_attn_fwd_f32(const AttnArgs& a, hipStream_t s) {
  ProfScope ps("attn_fwd_f32", s);
  launch_widths(a, [&](auto nc_, auto full_) {
    hipLaunchKernelGGL((attn_fwd_f32_kernel<decltype(nc_)::value, decltype(full_)::value>), dim3((a.S + AT - 1) / AT, a.H, a.B), dim3(64 * AW), 0, s, a);
  });
}

void launch_attn_bwd_f32(const AttnArgs& a, hipStream_t s) {
  ProfScope ps("attn_bwd_f32", s);
  const int n_dq = ((a.S + AT - 1) / AT) * a.H * a.B, n_dkv = ((a.L + AT - 1) / AT) * a.G * a.B;
  launch_widths(a, [&](auto nc_, auto full_) {
    hipLaunchKernelGGL((attn_bwd_f32_kernel<decltype(nc_)::value, decltype(full_)::value>), dim3(n_dq + n_dkv), dim3(64 * AW), 0, s, a, n_dq);
  });
}

}  // namespace beagle
