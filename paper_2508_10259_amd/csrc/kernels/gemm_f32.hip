// Projections of fp32 models: y = u W^T in full fp32 on the matrix cores
// (v_mfma_f32_16x16x4_f32: fp32 inputs, fp32 accumulation, 64 FLOP per clock
// and SIMD), with the epilogues of the fp16 GEMMs.
//
// An MFMA step takes 4 values of k, one per lane group g = lane / 16.  Both
// operands load 16 bytes (4 consecutive k) per lane and issue four steps from
// them, step e using element e of every group's four: any assignment of k to
// (step, group) is right as long as both operands share it, and no shuffles or
// 4-byte loads are needed.
#include "common.h"
#include "kernels.h"

namespace ams {

// ----------------------------------------------------------------------------
// M <= 64 tokens (decode passes, short token passes): bound by the weights,
// which are read once, and for small models by the launch itself.  A workgroup
// owns a strip of 16 packed weight rows (32 for SwiGLU: 16 gate + 16 up) on the
// M side of the MFMA, the tokens are its 1..4 column blocks, and up to 16 waves
// split K in chunks of 64 and meet in LDS, so even a 1 MB projection has
// thousands of loads in flight.  NRM (STORE, SWIGLU): the input is the residual stream itself;
// the sums of squares come from the activation fragments and 1/rms scales the
// result, which saves the separate norm launch (4.5 us each).
//
// gridDim.y > 1 (residual projections): the K range is cut in splits whose
// partial sums go out with device-scope stores; the last split of a strip to
// finish adds them in split order, so the result does not depend on arrival.
//
// Measured against 64 x 64 FMA tiles for every token count, us per launch.  One
// row, d = 256, FFN 1024: O and down 54.5 on average -> 3.1 and 4.7, QKV 23.5 ->
// 3.5, gate|up 23.1 -> 4.4.  Four rows, d = 1024, FFN 4096: O and down 298 on
// average -> 6.0 and 9.0, gate|up 125 -> 9.5 (3.5 TB/s), QKV 123 -> 6.6.  64
// tokens: O and down 298 -> 12.9 and 17.9, gate|up 125 -> 21.5.
struct GemvF32Args {
  const float* x;  // [M][K]
  const float* W;  // [N][K]
  float eps;
  int M, N, K;
  float* out;
  int ldo;
  float* part;    // gridDim.y > 1: [splits][M][N]
  unsigned* cnt;  // gridDim.y > 1: arrival counters per strip, zero between launches
};

template <int MB> constexpr int gemv_f32_waves() { return MB == 1 ? 16 : 8; }

template <int RB, int MB, int EPI>
__global__ __launch_bounds__((64 * gemv_f32_waves<MB>())) void k_gemv_f32(GemvF32Args a) {
  constexpr bool NRM = EPI != EPI_RESID;
  extern __shared__ __attribute__((aligned(16))) float red[];  // [nw][RB][MB][64 lanes][4], then (NRM) wsum[nw][MB*16], rstd[MB*16]
  __shared__ int last;
  const int tid = threadIdx.x, lane = tid & 63, nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int n0 = blockIdx.x * (RB * 16), M = a.M, K = a.K;
  const int nch = K >> 6, S = gridDim.y, sp = blockIdx.y;
  const int s0 = sp * nch / S, s1 = (sp + 1) * nch / S;
  const int c0 = s0 + wave * (s1 - s0) / nw, c1 = s0 + (wave + 1) * (s1 - s0) / nw;

  f32x4 acc[RB][MB];
#pragma unroll
  for (int q = 0; q < RB; ++q)
#pragma unroll
    for (int b = 0; b < MB; ++b) acc[q][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float* wrow[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) wrow[rb] = a.W + (size_t)(n0 + rb * 16 + r) * K + 4 * g;
  const float* xrow[MB];  // tokens >= M read token 0: they feed columns that are never stored
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int tok = mb * 16 + r;
    xrow[mb] = a.x + (size_t)(tok < M ? tok : 0) * K + 4 * g;
  }
  float ss[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) ss[mb] = 0.f;

  for (int c = c0; c < c1; ++c) {
    const int kb = c << 6;
    f32x4 fw[RB][4], fx[MB][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) fw[rb][i] = *(const f32x4*)(wrow[rb] + kb + 16 * i);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) fx[mb][i] = *(const f32x4*)(xrow[mb] + kb + 16 * i);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          const float xv = fx[mb][i][e];
          if constexpr (NRM) ss[mb] = fmaf(xv, xv, ss[mb]);
#pragma unroll
          for (int rb = 0; rb < RB; ++rb)
            acc[rb][mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[rb][i][e], xv, acc[rb][mb], 0, 0, 0);
        }
  }

#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      *(f32x4*)(red + (((wave * RB + rb) * MB + mb) * 64 + lane) * 4) = acc[rb][mb];
  float* wsum = red + (size_t)nw * RB * MB * 256;
  float* rstd = wsum + nw * MB * 16;
  if constexpr (NRM) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      float t = ss[mb];
      t += __shfl_xor(t, 16, 64);
      t += __shfl_xor(t, 32, 64);
      if (lane < 16) wsum[(wave * MB + mb) * 16 + lane] = t;
    }
    __syncthreads();
    if (tid < MB * 16) {
      float t = 0.f;
      for (int w = 0; w < nw; ++w) t += wsum[w * MB * 16 + tid];
      rstd[tid] = 1.0f / sqrtf(t / (float)K + a.eps);
    }
  }
  __syncthreads();

  // value (rb, mb, ln, i): packed row n0 + rb*16 + 4*(ln >> 4) + i, token mb*16 + (ln & 15)
  auto reduced = [&](int rb, int idx) {
    float t = 0.f;
    for (int w = 0; w < nw; ++w) t += red[((w * RB + rb) * MB) * 256 + idx];
    return t;
  };
  bool fin = true;
  if (EPI == EPI_RESID && S > 1) {
    for (int idx = tid; idx < MB * 256; idx += blockDim.x) {
      const int tok = (idx >> 8) * 16 + ((idx >> 2) & 15), row = 4 * ((idx >> 6) & 3) + (idx & 3);
      if (tok < M)
        __hip_atomic_store(a.part + ((size_t)sp * M + tok) * a.N + n0 + row, reduced(0, idx), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this thread's partial sums are stored
    __syncthreads();
    if (tid == 0) {
      unsigned* c = a.cnt + blockIdx.x;
      const bool l = __hip_atomic_fetch_add(c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(S - 1);
      if (l) __hip_atomic_store(c, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // every split is in
      last = l;
    }
    __syncthreads();
    fin = last != 0;
  }
  if (!fin) return;
  for (int idx = tid; idx < MB * 256; idx += blockDim.x) {
    const int tok = (idx >> 8) * 16 + ((idx >> 2) & 15), row = 4 * ((idx >> 6) & 3) + (idx & 3);
    if (tok >= M) continue;
    const float sc = NRM ? rstd[tok] : 1.f;
    if constexpr (EPI == EPI_SWIGLU) {  // the strip's first 16 rows are gate rows, the next 16 the up rows
      const float gt = reduced(0, idx) * sc, up = reduced(RB - 1, idx) * sc;
      a.out[(size_t)tok * a.ldo + (n0 >> 1) + row] = silu(gt) * up;
    } else {
      float* p = a.out + (size_t)tok * a.ldo + n0 + row;
      float y;
      if (EPI == EPI_RESID && S > 1) {
        y = 0.f;
        for (int s = 0; s < S; ++s)
          y += __hip_atomic_load(a.part + ((size_t)s * M + tok) * a.N + n0 + row, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
      } else {
        y = reduced(0, idx);
      }
      if constexpr (EPI == EPI_RESID) *p += y;
      else *p = y * sc;
    }
  }
}

template <int RB, int MB, int EPI>
static hipError_t launch_gemv_f32(const GemvF32Args& a, int splits, hipStream_t s) {
  const int nch = (a.K >> 6) / splits;
  int nw = gemv_f32_waves<MB>();
  while (nw > 1 && nw > nch) nw >>= 1;  // at least one chunk per wave
  const size_t lds = (size_t)nw * RB * MB * 1024 + (EPI != EPI_RESID ? (size_t)(nw + 1) * MB * 64 : 0);
  hipLaunchKernelGGL((k_gemv_f32<RB, MB, EPI>), dim3(a.N / (RB * 16), splits), dim3(64 * nw), lds, s, a);
  return hipGetLastError();
}

template <int EPI>
static hipError_t gemv_f32_m(const GemvF32Args& a, int splits, hipStream_t s) {
  constexpr int RB = EPI == EPI_SWIGLU ? 2 : 1;
  if (a.M <= 16) return launch_gemv_f32<RB, 1, EPI>(a, splits, s);
  if (a.M <= 32) return launch_gemv_f32<RB, 2, EPI>(a, splits, s);
  return launch_gemv_f32<RB, 4, EPI>(a, splits, s);
}

hipError_t gemv_f32(int epi, const float* x, bool norm, float eps, const float* W, int M, int N, int K, float* out,
                    int ldo, hipStream_t s, int splits, float* part, unsigned* cnt) {
  if (M <= 0) return hipSuccess;
  if (M > 64 || K % 64 != 0 || N % (epi == EPI_SWIGLU ? 32 : 16) != 0) return hipErrorInvalidValue;
  if (norm != (epi != EPI_RESID) || splits < 1 || splits > K / 64 ||
      (splits > 1 && (epi != EPI_RESID || !part || !cnt)))
    return hipErrorInvalidValue;
  const GemvF32Args a{x, W, eps, M, N, K, out, ldo, part, cnt};
  switch (epi) {
    case EPI_STORE: return gemv_f32_m<EPI_STORE>(a, 1, s);
    case EPI_RESID: return gemv_f32_m<EPI_RESID>(a, splits, s);
    default: return gemv_f32_m<EPI_SWIGLU>(a, 1, s);
  }
}

// ----------------------------------------------------------------------------
// Any M (the engine: more than 64): MFMA tiles of T x T (T = 128 or 64), four waves of T/2 x T/2, K steps
// of BK staged through registers into double-buffered LDS.  Bound by the MFMA
// rate: a step's arithmetic (2,048 cycles of a SIMD at T = 128) covers its
// loads.  Rows are padded to 96 or 160 bytes, pitches at which the 16-byte
// fragment reads are free of bank conflicts.  Against the 64 x 64 x 16 FMA tiles
// before it, at 1,200 tokens of d = 1024, FFN 4096: gate|up 387 -> 216 us (93
// TFLOP/s), QKV 192 -> 85 us, O and down 320 -> 106 us on average.

template <int EPI, int T, int BK>
__global__ __launch_bounds__(256) void k_gemm_f32(const float* __restrict__ u, const float* __restrict__ W, int M,
                                                  int K, float* __restrict__ out, int ldo) {
  constexpr int LDK = BK + 8, WT = T / 2, NB = WT / 16, CPR = BK / 4;  // LDS pitch, wave tile, chunks per row
  constexpr int LPT = T * CPR / 256;                                   // 16-byte loads per thread and operand
  __shared__ __attribute__((aligned(16))) float sm[2 * 2 * T * LDK];
  float* As = sm;                // [2][T][LDK]
  float* Bs = sm + 2 * T * LDK;  // [2][T][LDK]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane & 15, g = lane >> 4;
  const int wm = wave >> 1, wn = wave & 1;
  const int m0 = blockIdx.y * T, n0 = blockIdx.x * T;
  f32x4 ra[LPT], rb[LPT];
  auto load = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < LPT; ++q) {
      const int c = tid + 256 * q, row = c / CPR, kc = 4 * (c % CPR);
      const int ar = m0 + row < M ? m0 + row : M - 1;  // rows past M feed outputs that are never stored
      ra[q] = *(const f32x4*)(u + (size_t)ar * K + k0 + kc);
      rb[q] = *(const f32x4*)(W + (size_t)(n0 + row) * K + k0 + kc);
    }
  };
  auto stage = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < LPT; ++q) {
      const int c = tid + 256 * q, row = c / CPR, kc = 4 * (c % CPR);
      *(f32x4*)(As + (buf * T + row) * LDK + kc) = ra[q];
      *(f32x4*)(Bs + (buf * T + row) * LDK + kc) = rb[q];
    }
  };
  f32x4 acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int KT = K / BK;
  load(0);
  stage(0);
  __syncthreads();
  for (int kt = 0; kt < KT; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < KT) load((kt + 1) * BK);
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      f32x4 af[NB], bf[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i)
        af[i] = *(const f32x4*)(As + (cur * T + wm * WT + 16 * i + r) * LDK + 16 * ks + 4 * g);
#pragma unroll
      for (int j = 0; j < NB; ++j)
        bf[j] = *(const f32x4*)(Bs + (cur * T + wn * WT + 16 * j + r) * LDK + 16 * ks + 4 * g);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[i][e], bf[j][e], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < KT) stage(cur ^ 1);
    __syncthreads();
  }
  // block (i, j): lane holds tokens 4g + e of weight row r
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int tok = m0 + wm * WT + 16 * i + 4 * g + e;
      if (tok >= M) continue;
      if constexpr (EPI == EPI_SWIGLU) {  // blocks 2p (gate) and 2p + 1 (up) of the packed interleave
#pragma unroll
        for (int p = 0; p < NB / 2; ++p)
          out[(size_t)tok * ldo + ((n0 + wn * WT) >> 1) + 16 * p + r] = silu(acc[i][2 * p][e]) * acc[i][2 * p + 1][e];
      } else {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          float* p = out + (size_t)tok * ldo + n0 + wn * WT + 16 * j + r;
          if constexpr (EPI == EPI_RESID) *p += acc[i][j][e];
          else *p = acc[i][j][e];
        }
      }
    }
}

// 128-wide tiles, or 64-wide ones where those take less time by rounds of one
// workgroup per CU times tile area (O and down at 1,200 tokens of d = 1024: 80
// wide tiles keep 80 CUs busy, 304 narrow ones all of them) or where N is not a
// multiple of 128.
template <int EPI>
static hipError_t gemm_f32_epi(const float* u, const float* W, int M, int N, int K, float* out, int ldo,
                               hipStream_t s) {
  const long t128 = (long)(N / 128) * ((M + 127) / 128), t64 = (long)(N / 64) * ((M + 63) / 64);
  if (N % 128 == 0 && (t128 + 255) / 256 * 4 <= (t64 + 255) / 256) {
    hipLaunchKernelGGL((k_gemm_f32<EPI, 128, 16>), dim3(N / 128, (M + 127) / 128), dim3(256), 0, s, u, W, M, K, out,
                       ldo);
  } else {
    hipLaunchKernelGGL((k_gemm_f32<EPI, 64, 32>), dim3(N / 64, (M + 63) / 64), dim3(256), 0, s, u, W, M, K, out, ldo);
  }
  return hipGetLastError();
}

hipError_t gemm_f32(int epi, const float* u, const float* W, int M, int N, int K, float* out, int ldo, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (N % 64 != 0 || K % 32 != 0) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_STORE: return gemm_f32_epi<EPI_STORE>(u, W, M, N, K, out, ldo, s);
    case EPI_RESID: return gemm_f32_epi<EPI_RESID>(u, W, M, N, K, out, ldo, s);
    default: return gemm_f32_epi<EPI_SWIGLU>(u, W, M, N, K, out, ldo, s);
  }
}

}  // namespace ams
