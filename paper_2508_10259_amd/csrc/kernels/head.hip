// Action head, last stage: the bin logits (the last n_bins rows of the output
// head, computed by the projection GEMV after the final RMSNorm) reduced by a
// wavefront-shuffle argmax with the lowest bin winning ties; outputs, and the
// fed-back bin's embedding as the next decode pass's input.  One workgroup
// per row.
#include "common.h"
#include "kernels.h"

namespace ams {

// 8 consecutive elements of the embedding table as floats
__device__ __forceinline__ void head_load8(const float* p, float* v) {
  const float4 a = *(const float4*)p, b = *(const float4*)(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void head_load8(const f16* p, float* v) {
  const half8 a = __builtin_bit_cast(half8, *(const uint4*)p);
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = (float)a[i];
}

// Argmax + outputs + feedback over precomputed bin logits (one workgroup per
// row).  Bound by its chain of round trips (logits, forced bin, embedding row):
// the row moves 8 elements per thread and load (one before: 9.0 -> 5.0 us at d = 4096).
// With ss it also leaves the row's sums of squares per 128 columns, so that the
// next projection divides by its rms as after a residual reduction and the pass
// starts without a norm kernel.
template <typename T>
__global__ __launch_bounds__(256) void k_argmax_feed(const float* __restrict__ logits, int ldl, const T* __restrict__ bin_embed,
                                                     int d, int n_bins, int A, int j, int32_t* __restrict__ out_tok,
                                                     float* __restrict__ out_logits, const int32_t* __restrict__ forced,
                                                     float* __restrict__ h, int feed, T* __restrict__ h16,
                                                     T* __restrict__ h16lo, float* __restrict__ ss) {
  __shared__ float red[16];
  __shared__ int redi[16];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
  const float* lg = logits + (size_t)b * ldl;
  const size_t oj = (size_t)b * A + j;
  const int given = feed && forced ? forced[oj] : 0;  // in flight beside the logits
  float bv = -INFINITY;
  int bi = 0x7fffffff;
  for (int bin = tid; bin < n_bins; bin += blockDim.x) {
    const float v = lg[bin];
    if (out_logits) out_logits[oj * n_bins + bin] = v;
    if (v > bv) { bv = v; bi = bin; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(bv, o, 64);
    const int oi = __shfl_xor(bi, o, 64);
    if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
  }
  if (lane == 0) { red[wave] = bv; redi[wave] = bi; }
  __syncthreads();
  bv = red[0];
  bi = redi[0];
  for (int w = 1; w < nw; ++w)
    if (red[w] > bv || (red[w] == bv && redi[w] < bi)) { bv = red[w]; bi = redi[w]; }
  if (bi < 0 || bi >= n_bins) bi = 0;  // every logit NaN
  if (tid == 0) out_tok[oj] = bi;
  if (feed) {
    int t = forced ? given : bi;
    t = t < 0 ? 0 : (t >= n_bins ? n_bins - 1 : t);
    const T* e = bin_embed + (size_t)t * d;
    float* dst = h + (size_t)b * d;
    for (int i = 8 * tid; i < d; i += 8 * blockDim.x) {  // d is a multiple of 128: whole groups of 16 lanes
      float v[8];
      head_load8(e + i, v);
      *(float4*)(dst + i) = float4{v[0], v[1], v[2], v[3]};
      *(float4*)(dst + i + 4) = float4{v[4], v[5], v[6], v[7]};
      if (h16) {  // the embedding row is already in the compute type: its pair is (e, 0)
        *(uint4*)(h16 + (size_t)b * d + i) = *(const uint4*)(e + i);
        if (h16lo) *(uint4*)(h16lo + (size_t)b * d + i) = uint4{0u, 0u, 0u, 0u};
      }
      if (ss) {
        float q = 0.f;
#pragma unroll
        for (int x = 0; x < 8; ++x) q = fmaf(v[x], v[x], q);
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) q += __shfl_xor(q, o, 64);
        if ((lane & 15) == 0) ss[(size_t)b * (d / 128) + i / 128] = q;
      }
    }
  }
}

hipError_t argmax_feed(int ct, const float* logits, int ld_logits, const void* bin_embed, int B, int d, int n_bins,
                       int A, int j, int32_t* out_tok, float* out_logits, const int32_t* forced, float* h, int feed,
                       hipStream_t s, void* h16, void* h16lo, float* ss) {
  if (feed && d % 128 != 0) return hipErrorInvalidValue;
  if (ct == DT_F32) {
    if (h16 || h16lo || ss) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_argmax_feed<float>, dim3(B), dim3(256), 0, s, logits, ld_logits, (const float*)bin_embed, d,
                       n_bins, A, j, out_tok, out_logits, forced, h, feed, (float*)nullptr, (float*)nullptr, ss);
  } else {
    if (h16lo && !h16) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_argmax_feed<f16>, dim3(B), dim3(256), 0, s, logits, ld_logits, (const f16*)bin_embed, d,
                       n_bins, A, j, out_tok, out_logits, forced, h, feed, (f16*)h16, (f16*)h16lo, ss);
  }
  return hipGetLastError();
}

}  // namespace ams
