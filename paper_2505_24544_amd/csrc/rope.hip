// Rotary position embedding of projected queries / keys, in place (optional;
// section 4.1 leaves positional embeddings out of its equations, the LLaMA /
// Vicuna targets rotate Q and K).  Rotate-half convention: channel c < d/2 of a
// head is paired with channel c + d/2, angle = position * base^(-2c/d); the
// inverse rotation (the transpose) is what the backward pass applies to dQ, dK.
//
// Streaming kernels (bound: HBM): one workgroup per row (all heads of one
// position), the angles evaluated in double once per row.  Up to three tensors
// share one launch.
#include "common.h"

namespace beagle {
namespace {

// the tensor and row that a block owns, and the row's sequence position
__device__ __forceinline__ int locate_row(const RopeArgs& r, int64_t& row, int& pos) {
  int seg = 0;
  while (seg + 1 < r.n && row >= r.rows[seg]) { row -= r.rows[seg]; ++seg; }
  int idx = (int)(row % r.period[seg]);
  if (r.cu[seg]) {                               // packed batch: the entry whose rows include this one
    const int32_t* cu = r.cu[seg];
    int lo = 0, hi = r.nb;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (cu[mid] <= row) lo = mid; else hi = mid;
    }
    idx = (int)(row - cu[lo]);
  }
  pos = r.pos[seg] ? r.pos[seg][idx] : r.pos0[seg] + idx;
  return seg;
}

// float: any head width.  A thread owns two adjacent channel pairs of every eighth head.
__global__ __launch_bounds__(256) void rope_f32_kernel(RopeArgs r) {
  int64_t row = blockIdx.x;
  int pos;
  const int seg = locate_row(r, row, pos);
  const int d = r.d, half = d >> 1;
  const int c = 2 * (threadIdx.x % 32), hg = threadIdx.x / 32;   // first channel of this thread, head group
  if (c >= half) return;
  const float2 t0 = rope_cos_sin(pos, c, d, r.l2base), t1 = rope_cos_sin(pos, c + 1, d, r.l2base);
  const float fs0 = r.inverse ? -t0.y : t0.y, fs1 = r.inverse ? -t1.y : t1.y;
  float* x = (float*)r.x[seg] + row * (int64_t)r.heads[seg] * d;
  for (int h = hg; h < r.heads[seg]; h += 8) {
    float* p = x + h * d + c;
    const float2 a = *(const float2*)p, b = *(const float2*)(p + half);
    *(float2*)p = make_float2(a.x * t0.x - b.x * fs0, a.y * t1.x - b.y * fs1);
    *(float2*)(p + half) = make_float2(b.x * t0.x + a.x * fs0, b.y * t1.x + a.y * fs1);
  }
}

// bf16, head width 128: a thread owns eight channel pairs of a head in 16-byte accesses (32 heads per pass), the row's 64
// angles are evaluated by one wavefront while the rows travel.  Three tensors of 3048 rows x 32 heads (150 MB through): 28 us;
// with 4-byte accesses and the library's double sincos in every thread 40.
__global__ __launch_bounds__(256) void rope_bf16_kernel(RopeArgs r) {
  __shared__ float2 cs[64];
  int64_t row = blockIdx.x;
  int pos;
  const int seg = locate_row(r, row, pos);
  const int tid = threadIdx.x, c = 8 * (tid & 7), heads = r.heads[seg];
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  bf16_t* x = (bf16_t*)r.x[seg] + (row * heads + (tid >> 3)) * 128 + c;
  u32x4 a = {0, 0, 0, 0}, b = a;
  if ((tid >> 3) < heads) { a = *(const u32x4*)x; b = *(const u32x4*)(x + 64); }
  if (tid < 64) {
    float2 t = rope_cos_sin(pos, tid, 128, r.l2base);
    if (r.inverse) t.y = -t.y;
    cs[tid] = t;
  }
  __syncthreads();
  float2 t[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) t[i] = cs[c + i];
  for (int h = tid >> 3; h < heads; h += 32, x += 32 * 128) {
    if (h >= 32) { a = *(const u32x4*)x; b = *(const u32x4*)(x + 64); }
    u32x4 oa, ob;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float a0 = __uint_as_float(a[i] << 16), a1 = __uint_as_float(a[i] & 0xffff0000u);
      const float b0 = __uint_as_float(b[i] << 16), b1 = __uint_as_float(b[i] & 0xffff0000u);
      const float2 u = t[2 * i], v = t[2 * i + 1];
      oa[i] = pack_bf16x2(a0 * u.x - b0 * u.y, a1 * v.x - b1 * v.y);
      ob[i] = pack_bf16x2(b0 * u.x + a0 * u.y, b1 * v.x + a1 * v.y);
    }
    *(u32x4*)x = oa;
    *(u32x4*)(x + 64) = ob;
  }
}

}  // namespace

void launch_rope(bool bf16, const RopeArgs& r, hipStream_t s, const char* name) {
  int64_t total = 0;
  for (int i = 0; i < r.n; ++i) total += r.rows[i];
  if (total == 0) return;
  ProfScope ps(name, s);
  if (bf16) hipLaunchKernelGGL(rope_bf16_kernel, dim3((unsigned)total), dim3(256), 0, s, r);   // (bf16 storage: head width 128)
  else hipLaunchKernelGGL(rope_f32_kernel, dim3((unsigned)total), dim3(256), 0, s, r);
}

}  // namespace beagle
