// Late-stage simulation (section 4.2, second half) in float: the band of
// predicted keys as plain FMA code, one wavefront per row (bf16 storage:
// sim_band_bf16.hip), and the in-place save of predicted states.
#include "common.h"

namespace beagle {

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// --------------------------------------------------------------------------
// Late-stage simulation (section 4.2, second half): every query also sees the
// predicted states of at most t earlier positions of its own window.  That
// band is a handful of keys per query, so it runs as plain FMA code, one
// wavefront per query row (forward, dQ) or per predicted key row (dKp, dVp),
// lanes owning head channels:
//   forward : (O, LSE) of the masked attention over the true keys is merged
//             with the band: LSE' = logaddexp(LSE, lse_band), O' the weighted mean;
//   backward: the main kernels, given LSE' and delta = rowsum(dO * O'), already
//             produce the true-key parts; the band adds its share to dQ and
//             yields dKp, dVp (zero on rows that no query sees).
// --------------------------------------------------------------------------
__global__ __launch_bounds__(64) void sim_band_fwd_kernel(SimArgs s) {
  const AttnArgs& a = s.a;
  const int p = blockIdx.x, h = blockIdx.y, b = blockIdx.z, lane = threadIdx.x;
  const SeqView sv = seq_view(a, b);
  if (p >= sv.S) return;                               // packed batch: a shorter entry
  int lo, hi;
  sim_band(p, a.mask.k, sample_mask(a, b).eps, s.t, sv.L, lo, hi);
  if (hi <= lo) return;
  const int d = a.d, g = h / (a.H / a.G);
  const int64_t kvs = (int64_t)a.G * d;
  const float* Q = (const float*)a.q + ((sv.q0 + p) * a.H + h) * d;
  float* O = (float*)a.o + ((sv.q0 + p) * a.H + h) * d;
  const float* Kp = (const float*)s.kp + (sv.kv0 * a.G + g) * d;
  const float* Vp = (const float*)s.vp + (sv.kv0 * a.G + g) * d;
  const int64_t li = sv.lse0 + h * sv.lse_hs + p;
  const bool c0 = lane < d, c1 = lane + 64 < d;
  const float q0 = c0 ? Q[lane] : 0.f, q1 = c1 ? Q[lane + 64] : 0.f;
  float m = a.lse[li];                                   // weight of the true-key part: exp(m) * 1
  float l = m > -INFINITY ? 1.f : 0.f;
  float acc0 = (c0 && l > 0.f) ? O[lane] : 0.f, acc1 = (c1 && l > 0.f) ? O[lane + 64] : 0.f;
  for (int j = lo; j < hi; ++j) {
    const float* kr = Kp + j * kvs;
    const float* vr = Vp + j * kvs;
    const float sc = a.scale * wave_sum((c0 ? q0 * kr[lane] : 0.f) + (c1 ? q1 * kr[lane + 64] : 0.f));
    const float mn = fmaxf(m, sc);
    const float al = expf(m - mn), pj = expf(sc - mn);   // m = -inf: al = 0
    acc0 = acc0 * al + (c0 ? pj * vr[lane] : 0.f);
    acc1 = acc1 * al + (c1 ? pj * vr[lane + 64] : 0.f);
    l = l * al + pj;
    m = mn;
  }
  const float inv = 1.f / l;
  if (c0) O[lane] = acc0 * inv;
  if (c1) O[lane + 64] = acc1 * inv;
  if (lane == 0) a.lse[li] = m + logf(l);
}

__global__ __launch_bounds__(64) void sim_band_bwd_dq_kernel(SimArgs s) {
  const AttnArgs& a = s.a;
  const int p = blockIdx.x, h = blockIdx.y, b = blockIdx.z, lane = threadIdx.x;
  const SeqView sv = seq_view(a, b);
  if (p >= sv.S) return;                               // packed batch: a shorter entry
  int lo, hi;
  sim_band(p, a.mask.k, sample_mask(a, b).eps, s.t, sv.L, lo, hi);
  if (hi <= lo) return;
  const int d = a.d, g = h / (a.H / a.G);
  const int64_t kvs = (int64_t)a.G * d;
  const int64_t row = ((sv.q0 + p) * a.H + h) * d;
  const float* Q = (const float*)a.q + row;
  const float* dO = (const float*)a.dout + row;
  float* dQ = (float*)a.dq + row;
  const float* Kp = (const float*)s.kp + (sv.kv0 * a.G + g) * d;
  const float* Vp = (const float*)s.vp + (sv.kv0 * a.G + g) * d;
  const int64_t li = sv.lse0 + h * sv.lse_hs + p;
  const bool c0 = lane < d, c1 = lane + 64 < d;
  const float q0 = c0 ? Q[lane] : 0.f, q1 = c1 ? Q[lane + 64] : 0.f;
  const float g0 = c0 ? dO[lane] : 0.f, g1 = c1 ? dO[lane + 64] : 0.f;
  const float lse = a.lse[li], delta = a.delta[li];
  float a0 = 0.f, a1 = 0.f;
  for (int j = lo; j < hi; ++j) {
    const float* kr = Kp + j * kvs;
    const float* vr = Vp + j * kvs;
    const float k0 = c0 ? kr[lane] : 0.f, k1 = c1 ? kr[lane + 64] : 0.f;
    const float v0 = c0 ? vr[lane] : 0.f, v1 = c1 ? vr[lane + 64] : 0.f;
    const float pj = expf(a.scale * wave_sum(q0 * k0 + q1 * k1) - lse);
    const float ds = pj * (wave_sum(g0 * v0 + g1 * v1) - delta);
    a0 = fmaf(ds, k0, a0);
    a1 = fmaf(ds, k1, a1);
  }
  if (c0) dQ[lane] = dQ[lane] + a0 * a.scale;
  if (c1) dQ[lane + 64] = dQ[lane + 64] + a1 * a.scale;
}

__global__ __launch_bounds__(64) void sim_band_bwd_dkv_kernel(SimArgs s) {
  const AttnArgs& a = s.a;
  const int j = blockIdx.x, g = blockIdx.y, b = blockIdx.z, lane = threadIdx.x;
  const SeqView sv = seq_view(a, b);
  if (j >= sv.L) return;                               // packed batch: a shorter entry
  const int d = a.d, rep = a.H / a.G;
  const int64_t kvrow = ((sv.kv0 + j) * a.G + g) * d;
  const float* kr = (const float*)s.kp + kvrow;
  const float* vr = (const float*)s.vp + kvrow;
  const bool c0 = lane < d, c1 = lane + 64 < d;
  float dk0 = 0.f, dk1 = 0.f, dv0 = 0.f, dv1 = 0.f;
  const int w0 = window_start_raw(j, a.mask.k, sample_mask(a, b).eps);
  if (j - w0 < s.t) {                                  // this position holds a predicted state at step t
    const float k0 = c0 ? kr[lane] : 0.f, k1 = c1 ? kr[lane + 64] : 0.f;
    const float v0 = c0 ? vr[lane] : 0.f, v1 = c1 ? vr[lane + 64] : 0.f;
    const int p_end = min(w0 + a.mask.k, sv.S);         // the later queries of the same window see it
    for (int p = j + 1; p < p_end; ++p)
      for (int hh = 0; hh < rep; ++hh) {
        const int h = g * rep + hh;
        const int64_t row = ((sv.q0 + p) * a.H + h) * d;
        const float* Q = (const float*)a.q + row;
        const float* dO = (const float*)a.dout + row;
        const int64_t li = sv.lse0 + h * sv.lse_hs + p;
        const float q0 = c0 ? Q[lane] : 0.f, q1 = c1 ? Q[lane + 64] : 0.f;
        const float g0 = c0 ? dO[lane] : 0.f, g1 = c1 ? dO[lane + 64] : 0.f;
        const float pj = expf(a.scale * wave_sum(q0 * k0 + q1 * k1) - a.lse[li]);
        const float ds = pj * (wave_sum(g0 * v0 + g1 * v1) - a.delta[li]);
        dk0 = fmaf(ds, q0, dk0); dk1 = fmaf(ds, q1, dk1);
        dv0 = fmaf(pj, g0, dv0); dv1 = fmaf(pj, g1, dv1);
      }
  }
  float* dK = (float*)s.dkp + kvrow;
  float* dV = (float*)s.dvp + kvrow;
  if (c0) { dK[lane] = dk0 * a.scale; dV[lane] = dv0; }
  if (c1) { dK[lane + 64] = dk1 * a.scale; dV[lane + 64] = dv1; }
}

void launch_sim_band_fwd(const SimArgs& s, hipStream_t st) {
  if (s.is_bf16) return launch_sim_band_fwd_bf16(s, st);    // bf16 storage implies head width 128
  ProfScope ps("sim_band_fwd", st);
  dim3 grid(s.a.S, s.a.H, s.a.B);
  hipLaunchKernelGGL(sim_band_fwd_kernel, grid, dim3(64), 0, st, s);
}
void launch_sim_band_bwd(const SimArgs& s, hipStream_t st) {
  if (s.is_bf16) return launch_sim_band_bwd_bf16(s, st);
  {
    ProfScope ps("sim_band_bwd_dq", st);
    dim3 grid(s.a.S, s.a.H, s.a.B);
    hipLaunchKernelGGL(sim_band_bwd_dq_kernel, grid, dim3(64), 0, st, s);
  }
  {
    ProfScope ps("sim_band_bwd_dkv", st);
    dim3 grid(s.a.L, s.a.G, s.a.B);
    hipLaunchKernelGGL(sim_band_bwd_dkv_kernel, grid, dim3(64), 0, st, s);
  }
}

// In-place update of the predicted-state buffer between simulation steps (section 4.2, second half):
// after step t the row at position t of every window takes the newly predicted state of that position.
// blockIdx.x: window (the partial leading one first), blockIdx.y: batch entry; rows as 16-byte chunks.
__global__ __launch_bounds__(256) void sim_save_kernel(const uint4* __restrict__ h, uint4* __restrict__ xpred, int L,
                                                       int chunks, int k, int eps, const int32_t* eps_b, int t,
                                                       const int32_t* cu, int total) {
  if (eps_b) { eps = eps_b[blockIdx.y] % k; if (eps < 0) eps += k; }
  int64_t first = (int64_t)blockIdx.y * L;          // first row of this entry
  if (cu) {                                          // packed batch: clamped like the attention kernels' view
    const int32_t r0 = min(max(cu[blockIdx.y], 0), total);
    L = min(max(cu[blockIdx.y + 1] - r0, 0), min(L, total - r0));
    first = r0;
  }
  const int n0 = eps > 0 ? eps - k : 0;
  const int j = n0 + (int)blockIdx.x * k + t;
  if (j < 0 || j >= L) return;
  const int64_t row = (first + j) * chunks;
  for (int c = threadIdx.x; c < chunks; c += 256) xpred[row + c] = h[row + c];
}

void launch_sim_save(const void* h, void* xpred, int B, int L, int64_t row_bytes, int k, int eps, const int32_t* eps_b,
                     int t, const int32_t* cu, int total, hipStream_t st) {
  ProfScope ps("sim_save", st);
  const int n0 = (eps_b || eps > 0) ? -k + 1 : 0;   // lowest possible start of the leading window
  const int n_win = (L - n0 + k - 1) / k + 1;
  hipLaunchKernelGGL(sim_save_kernel, dim3(n_win, B), dim3(256), 0, st, (const uint4*)h, (uint4*)xpred, L,
                     (int)(row_bytes / 16), k, eps, eps_b, t, cu, total);
}

}  // namespace beagle
