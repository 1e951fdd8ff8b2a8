// Flow-matching action head over a cached context (paper section 3.2.1: the
// diffusion model's latent vectors are part of the action context; section
// 3.4.2, Action Regeneration: sampling restarts from a stored latent).
//
// One Euler step of the latent x [token][a] of every row's action chunk:
//   k_flow_embed:  h[t] = W_in x[t] + tau w_t      (the chunk's tokens enter the decoder)
//   (every decoder layer over the tokens, at the positions after each row's context)
//   k_flow_update: x[t] += dt W_out (h[t] / rms(h[t]))
// Both are small per-token kernels around the decoder's token pass; the pass
// itself (GEMMs on MFMA, attention over the cached K/V pages) is the same code
// that builds and extends contexts.
#include "common.h"
#include "kernels.h"

namespace ams {

namespace {

// 256 output dimensions (one per thread) of EMBED_TOK tokens: a thread's weight
// row is read once for all of them, the tokens' values come from LDS.  Bound by
// the launch at the sizes of an action chunk (128 tokens of 7 values, d = 4096:
// one workgroup per token re-read the weights 2 bytes at a time, 34 -> 5 us).
constexpr int EMBED_TOK = 8;
template <typename T>
__global__ __launch_bounds__(256) void k_flow_embed(const float* __restrict__ x, const T* __restrict__ w_in,
                                                    const T* __restrict__ w_t, float tau, int n_tok, int a, int d,
                                                    float* __restrict__ h) {
  __shared__ float xs[EMBED_TOK * FLOW_MAX_ACTION_DIM];
  const int t0 = blockIdx.y * EMBED_TOK, nt = min(EMBED_TOK, n_tok - t0);
  for (int k = threadIdx.x; k < nt * a; k += blockDim.x) xs[k] = x[(size_t)t0 * a + k];
  __syncthreads();
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= d) return;
  float e[EMBED_TOK];
  const float e0 = tau * ld<T>(w_t, j);
#pragma unroll
  for (int t = 0; t < EMBED_TOK; ++t) e[t] = e0;
  for (int k = 0; k < a; ++k) {
    const float w = ld<T>(w_in, (size_t)j * a + k);
#pragma unroll
    for (int t = 0; t < EMBED_TOK; ++t) e[t] = fmaf(w, xs[min(t, nt - 1) * a + k], e[t]);
  }
#pragma unroll
  for (int t = 0; t < EMBED_TOK; ++t)
    if (t < nt) h[(size_t)(t0 + t) * d + j] = e[t];
}

// 8 consecutive weights as floats
__device__ __forceinline__ void flow_load8(const float* p, float* v) {
  const float4 a = *(const float4*)p, b = *(const float4*)(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void flow_load8(const bf16* p, float* v) {
  const uint4 q = *(const uint4*)p;
  const uint32_t u[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(u[i] << 16);
    v[2 * i + 1] = __uint_as_float(u[i] & 0xFFFF0000u);
  }
}

// One workgroup of 8 waves per token: its row of h goes to LDS with the sum of
// squares, then one output per wave at a time, 8 values per lane and load, and a
// wavefront sum (one 2-byte weight per lane and load before: 34 -> 5 us for 128
// tokens of d = 4096).  w_out is 16-byte aligned and d a multiple of 128 (VEC), or
// read element by element.
template <typename T, bool VEC>
__global__ __launch_bounds__(512) void k_flow_update(const float* __restrict__ h, const T* __restrict__ w_out,
                                                     float eps, float dt, int a, int d, float* __restrict__ x) {
  extern __shared__ __attribute__((aligned(16))) float hs[];  // [d]
  __shared__ float red[16];
  const int t = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const float* ht = h + (size_t)t * d;
  float ss = 0.f;
  for (int j = 4 * threadIdx.x; j < d; j += 4 * blockDim.x) {
    const float4 v = *(const float4*)(ht + j);
    *(float4*)(hs + j) = v;
    ss = fmaf(v.x, v.x, ss);
    ss = fmaf(v.y, v.y, ss);
    ss = fmaf(v.z, v.z, ss);
    ss = fmaf(v.w, v.w, ss);
  }
  const float r = rsqrtf(block_sum(ss, red) / (float)d + eps);  // (its barriers publish hs)
  for (int i = wave; i < a; i += nw) {
    const T* w = w_out + (size_t)i * d;
    float v = 0.f;
    if constexpr (VEC) {
      float v1 = 0.f;
#pragma unroll 4
      for (int j = 8 * lane; j < d; j += 512) {
        float wv[8];
        flow_load8(w + j, wv);
        const float4 a0 = *(const float4*)(hs + j), a1 = *(const float4*)(hs + j + 4);
        v = fmaf(wv[0], a0.x, v);
        v1 = fmaf(wv[1], a0.y, v1);
        v = fmaf(wv[2], a0.z, v);
        v1 = fmaf(wv[3], a0.w, v1);
        v = fmaf(wv[4], a1.x, v);
        v1 = fmaf(wv[5], a1.y, v1);
        v = fmaf(wv[6], a1.z, v);
        v1 = fmaf(wv[7], a1.w, v1);
      }
      v += v1;
    } else {
      for (int j = lane; j < d; j += 64) v = fmaf(ld<T>(w, j), hs[j], v);
    }
    v = wave_sum(v);
    if (lane == 0) x[(size_t)t * a + i] += dt * (v * r);
  }
}

}  // namespace

hipError_t flow_embed(int st, const float* x, const void* w_in, const void* w_t, float tau, int n_tok, int a, int d,
                      float* h, hipStream_t s) {
  if (n_tok <= 0) return hipSuccess;
  if (a < 1 || a > FLOW_MAX_ACTION_DIM) return hipErrorInvalidValue;
  const dim3 grid((d + 255) / 256, (n_tok + EMBED_TOK - 1) / EMBED_TOK);
  if (st == DT_F32)
    hipLaunchKernelGGL(k_flow_embed<float>, grid, dim3(256), 0, s, x, (const float*)w_in, (const float*)w_t, tau,
                       n_tok, a, d, h);
  else
    hipLaunchKernelGGL(k_flow_embed<bf16>, grid, dim3(256), 0, s, x, (const bf16*)w_in, (const bf16*)w_t, tau, n_tok,
                       a, d, h);
  return hipGetLastError();
}

hipError_t flow_update(int st, const float* h, const void* w_out, float eps, float dt, int n_tok, int a, int d,
                       float* x, hipStream_t s) {
  if (n_tok <= 0) return hipSuccess;
  const size_t lds = (size_t)d * 4;
  const bool vec = ((uintptr_t)w_out & 15) == 0;
#define AMS_FU(T, V) \
  hipLaunchKernelGGL((k_flow_update<T, V>), dim3(n_tok), dim3(512), lds, s, h, (const T*)w_out, eps, dt, a, d, x)
  if (st == DT_F32) {
    if (vec) AMS_FU(float, true);
    else AMS_FU(float, false);
  } else {
    if (vec) AMS_FU(bf16, true);
    else AMS_FU(bf16, false);
  }
#undef AMS_FU
  return hipGetLastError();
}

}  // namespace ams
