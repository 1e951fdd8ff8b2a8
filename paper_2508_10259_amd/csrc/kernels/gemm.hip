// Projection and feed-forward GEMMs: y = u W^T with fused epilogues.
//
//  * k_gemm_skinny  (fp16, M <= 64 tokens: the per-action decode pass of up to 8
//    rows outside the persistent kernel, and, on fragment-ordered weights, token passes
//    but those of 33 to 64 tokens on large weights).  HBM
//    bound on the weights: every weight byte is read exactly once.  A
//    workgroup owns a strip of 16 (or 32 for SwiGLU: 16 gate + 16 up) packed weight rows; its
//    waves split K in chunks of 128 and run v_mfma_f32_16x16x32_f16 with the
//    weight rows on the M side and up to 64 tokens as 1..4 column blocks, so a
//    weight fragment is loaded once and reused for every token block.  The
//    per-wave partial sums meet in LDS; the epilogue (store / residual add /
//    SiLU-gate) runs on the reduced values.  Up to 16 tokens it can also
//    apply the preceding RMSNorm itself (gemv_rmsnorm).  RMSNorm gains are
//    folded into the packed weights, so every GEMM consumes h / rms(h).
//  * k_gemm_wide    (fp16, batched decode of 9 to 64 rows, those token passes).
//  Longer token passes: gemm_tokens.hip.
//  fp32 models: gemm_f32.hip, same epilogues.
#include "common.h"
#include "kernels.h"

namespace ams {

__device__ __forceinline__ half8 as_half8(uint4 v) { return __builtin_bit_cast(half8, v); }
typedef _Float16 half2v __attribute__((ext_vector_type(2)));

// ----------------------------------------------------------------------------
// skinny: M <= 64
//
// Each wave requests the weight and activation fragments of up to CPW of its
// K chunks before the first MFMA, so its loads overlap in one round trip; a
// residual epilogue's h values are requested at kernel entry for the same
// reason.  The K range a wave covers is rotated by the workgroup index, so
// concurrent workgroups read different parts of the shared activations.
//
// Compensated input (LO != 0): the activations arrive as an fp16 pair
// x = hi + lo (lo = the rounding error of hi), and W x = W hi + W lo, so the
// product carries about 22 significant bits of x instead of 11.  With up to 8
// tokens (LO == 1) the pair shares one MFMA: B columns 0..7 take hi, columns
// 8..15 take lo of the same tokens, and the epilogue adds the two halves;
// otherwise (LO == 2) lo has its own fragments and MFMAs.
//
// NRM (M <= 16): the input is the (fp16 or fp16-pair) copy of the residual
// stream h [M][K] and the kernel applies RMSNorm itself: the MFMA consumes it
// as is, the sum of squares of each token row comes from the hi fragments
// (reduced across the waves, which together cover all of K), and the 1/rms
// scale multiplies the result in the epilogue.  The RMSNorm gain is folded
// into W at packing.  Taking the statistic from hi alone changes it by about
// 2^-11 / sqrt(K) relative for rounding errors of random sign (the product,
// where one term's error does not average out, takes hi + lo).
//
// RESID may also write the updated residual rows as fp16 (ohi, and olo for
// the pair), the input of the next fused-RMSNorm GEMV; SWIGLU may write the
// rounding error of its fp16 output to olo.

struct SkinnyArgs {
  const f16* xhi;  // [M][K]
  const f16* xlo;  // [M][K] or NULL
  float eps;
  const f16* W;    // [N][K]
  int M, K;
  void* out;
  int ldo;
  f16* ohi;  // RESID only, or NULL
  f16* olo;  // RESID / SWIGLU, or NULL
};

// most waves per workgroup: 16 for the SwiGLU strip with one token block (its
// two chunks in flight fit 128 VGPRs), 8 otherwise (256 VGPRs)
template <int RB, int MB, int LO>
constexpr int skinny_max_waves() {
  return RB == 2 && MB == 1 && LO != 2 ? 16 : 8;
}

template <int RB, int MB, int LO>
constexpr int skinny_cpw() {
  return (RB + MB * (LO == 2 ? 2 : 1)) <= 2 ? 4 : ((RB + MB * (LO == 2 ? 2 : 1)) <= 4 ? 2 : 1);
}

template <int RB, int MB, int EPI, bool NRM, int LO, bool FRAG>
__global__ __launch_bounds__((64 * skinny_max_waves<RB, MB, LO>())) void k_gemm_skinny(SkinnyArgs a) {
  static_assert(!NRM || MB == 1, "the fused RMSNorm handles up to 16 tokens");
  static_assert(!NRM || EPI != EPI_PART, "the RMS statistic needs all of K");
  static_assert(LO != 1 || MB == 1, "the packed pair handles up to 8 tokens");
  constexpr int LB = LO == 2 ? MB : 1;  // lo fragment blocks (unused unless LO == 2)
  extern __shared__ float red[];  // [nw][RB][MB][64 lanes][4], then (NRM) wsum[<=16 waves][16] + rstd[16]
  const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform: chunk loops branch on scalars
  const int r = lane & 15, g = lane >> 4;
  const int n0 = blockIdx.x * (RB * 16);
  const int M = a.M, K = a.K, ldo = a.ldo;
  // K chunks of this workgroup: split blockIdx.y of gridDim.y (EPI_PART), shared by the waves
  const int nchunks = K >> 7, S = gridDim.y, sp = blockIdx.y;
  const int s0 = sp * nchunks / S, s1 = (sp + 1) * nchunks / S;
  const int wk = (wave + blockIdx.x) % nw;
  const int c0 = s0 + wk * (s1 - s0) / nw, c1 = s0 + (wk + 1) * (s1 - s0) / nw;

  f32x4 acc[RB][MB];
#pragma unroll
  for (int q = 0; q < RB; ++q)
#pragma unroll
    for (int b = 0; b < MB; ++b) acc[q][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  const f16* wrow[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
    wrow[rb] = FRAG ? a.W + (size_t)(n0 + rb * 16) * K + lane * 8 : a.W + (size_t)(n0 + rb * 16 + r) * K + g * 8;
  constexpr int WS = FRAG ? 16 : 1;  // a lane's weights of 32 columns on: 1 KB block on, or 64 bytes
  // B-operand rows of this lane: token mb*16 + r (LO == 1: token r & 7, hi for r < 8, lo above).
  // Columns of tokens >= M read token 0 instead of being masked (a masked load
  // costs a branch per load): they only feed output columns that are never
  // stored, and statistics that are never read.
  const f16* urow[MB];
  const f16* lrow[LB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int tok = LO == 1 ? (r & 7) : mb * 16 + r;
    const size_t off = (size_t)(tok < M ? tok : 0) * K + g * 8;
    urow[mb] = (LO == 1 && r >= 8 ? a.xlo : a.xhi) + off;
    if constexpr (LO == 2) lrow[mb] = a.xlo + off;
  }
  float ss0 = 0.f, ss1 = 0.f;  // NRM: this lane's share of sum(x^2) of its token (two chains)

  // the residual epilogue's h values do not depend on this kernel: request them first
  constexpr int EPT = (MB * 256 + 63) / 64;  // epilogue values per thread at the smallest workgroup
  float hres[EPI == EPI_RESID ? RB * EPT : 1];
  if constexpr (EPI == EPI_RESID) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int idx = threadIdx.x + e * blockDim.x;
      const int mb = idx >> 8, ln = (idx >> 2) & 63, i = idx & 3;
      const int tok = mb * 16 + (ln & 15), row = 4 * (ln >> 4) + i;
      const bool ok = idx < MB * 256 && tok < M && (LO != 1 || (ln & 15) < 8);
      const size_t at = (size_t)(ok ? tok : 0) * ldo + n0 + row;  // unused values read row 0
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) hres[rb * EPT + e] = ((const float*)a.out)[at + rb * 16];
    }
  }

  // chunks in flight per wave: up to CPW loads are issued before the first MFMA
  constexpr int CPW = skinny_cpw<RB, MB, LO>();
  uint4 fw[CPW][RB][4], fu[CPW][MB][4], fl[CPW][LB][4];
  for (int cb = c0; cb < c1; cb += CPW) {
#pragma unroll
    for (int j = 0; j < CPW; ++j) {
      if (cb + j < c1) {
        const int kb = (cb + j) << 7;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int i = 0; i < 4; ++i) fw[j][rb][i] = ld_stream(wrow[rb] + (kb + 32 * i) * WS);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            fu[j][mb][i] = *(const uint4*)(urow[mb] + kb + 32 * i);
            if constexpr (LO == 2) fl[j][mb][i] = *(const uint4*)(lrow[mb] + kb + 32 * i);
          }
      }
    }
#pragma unroll
    for (int j = 0; j < CPW; ++j) {
      if (cb + j < c1) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const half8 v = as_half8(fu[j][mb][i]);
            if constexpr (NRM) {  // the statistic reads hi only (LO == 1: lanes r >= 8 are unused)
              const half2v* p2 = (const half2v*)&fu[j][mb][i];
              ss0 = __builtin_amdgcn_fdot2(p2[0], p2[0], ss0, false);
              ss1 = __builtin_amdgcn_fdot2(p2[1], p2[1], ss1, false);
              ss0 = __builtin_amdgcn_fdot2(p2[2], p2[2], ss0, false);
              ss1 = __builtin_amdgcn_fdot2(p2[3], p2[3], ss1, false);
            }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
              acc[rb][mb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(fw[j][rb][i]), v, acc[rb][mb], 0, 0, 0);
              if constexpr (LO == 2)
                acc[rb][mb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(fw[j][rb][i]), as_half8(fl[j][mb][i]),
                                                                      acc[rb][mb], 0, 0, 0);
            }
          }
      }
    }
  }

#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int i = 0; i < 4; ++i) red[(((wave * RB + rb) * MB + mb) * 64 + lane) * 4 + i] = acc[rb][mb][i];
  float* rstd = red + (size_t)nw * RB * MB * 256 + 256;
  if constexpr (NRM) {
    float* wsum = rstd - 256;  // [16 waves][16 tokens]
    float ss = ss0 + ss1;
    ss += __shfl_xor(ss, 16, 64);
    ss += __shfl_xor(ss, 32, 64);
    if (lane < 16) wsum[wave * 16 + lane] = ss;
    __syncthreads();
    if (threadIdx.x < 16) {
      float t = 0.f;
      for (int w = 0; w < nw; ++w) t += wsum[w * 16 + threadIdx.x];
      rstd[threadIdx.x] = 1.0f / sqrtf(t / (float)K + a.eps);
    }
  }
  __syncthreads();

  // value (rb, mb, ln, i) is packed row n0 + rb*16 + 4*(ln>>4) + i, B column mb*16 + (ln&15);
  // summed over the waves (and, LO == 1, over the hi and lo columns ln and ln+8)
  auto reduced = [&](int rb, int mb, int ln, int i) {
    float t = 0.f;
    for (int w = 0; w < nw; ++w) {
      t += red[(((w * RB + rb) * MB + mb) * 64 + ln) * 4 + i];
      if constexpr (LO == 1) t += red[(((w * RB + rb) * MB + mb) * 64 + ln + 8) * 4 + i];
    }
    return t;
  };
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const int idx = threadIdx.x + e * blockDim.x;
    if (idx >= MB * 256) break;
    const int mb = idx >> 8, ln = (idx >> 2) & 63, i = idx & 3;
    const int tok = mb * 16 + (ln & 15);
    if (tok >= M || (LO == 1 && (ln & 15) >= 8)) continue;
    const int row = 4 * (ln >> 4) + i;
    const float sc = NRM ? rstd[tok] : 1.f;
    if constexpr (EPI == EPI_STORE) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
        ((float*)a.out)[(size_t)tok * ldo + n0 + rb * 16 + row] = reduced(rb, mb, ln, i) * sc;
    } else if constexpr (EPI == EPI_PART) {  // this split's partial sums: out[sp][tok][n]
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
        ((float*)a.out)[((size_t)sp * M + tok) * ldo + n0 + rb * 16 + row] = reduced(rb, mb, ln, i);
    } else if constexpr (EPI == EPI_RESID) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const size_t o = (size_t)tok * ldo + n0 + rb * 16 + row;
        const float hn = hres[rb * EPT + e] + reduced(rb, mb, ln, i) * sc;
        ((float*)a.out)[o] = hn;
        if (a.ohi) split16(hn, a.ohi, a.olo, o);
      }
    } else {  // the strip's first 16 rows are gate rows, the next 16 the up rows of the same outputs
      const float gt = reduced(0, mb, ln, i) * sc, up = reduced(RB - 1, mb, ln, i) * sc;
      split16(silu(gt) * up, (f16*)a.out, a.olo, (size_t)tok * ldo + (n0 >> 1) + row);
    }
  }
}

template <int RB, int MB, int EPI, bool NRM, int LO, bool FRAG = false>
static hipError_t launch_skinny(const SkinnyArgs& a, int N, hipStream_t s, int splits = 1) {
  // waves per workgroup: at most 64 KB of reduction LDS and at least one chunk
  // per wave; the 16-wave variant takes 16 only when every wave then gets a
  // full batch of CPW chunks (all chunks go out in one round), 8 otherwise
  const int nchunks = (a.K >> 7) / splits;
  constexpr int MW = skinny_max_waves<RB, MB, LO>();
  int nw = MW == 16 && nchunks < 16 * skinny_cpw<RB, MB, LO>() ? 8 : MW;
  while (nw > 1 && nw * RB * MB * 1024 > 65536) nw >>= 1;
  while (nw > 1 && nw > nchunks) nw >>= 1;
  const size_t lds = (size_t)nw * RB * MB * 1024 + (NRM ? (256 + 16) * 4 : 0);
  hipLaunchKernelGGL((k_gemm_skinny<RB, MB, EPI, NRM, LO, FRAG>), dim3(N / (RB * 16), splits), dim3(64 * nw), lds, s, a);
  return hipGetLastError();
}

// token blocks and input form of one skinny launch
template <int EPI, bool NRM>
static hipError_t skinny_dispatch(const SkinnyArgs& a, int N, hipStream_t s) {
  constexpr int RB = EPI == EPI_SWIGLU ? 2 : 1;
  const int M = a.M;
  if (!a.xlo) {
    if (M <= 16) return launch_skinny<RB, 1, EPI, NRM, 0>(a, N, s);
    if constexpr (!NRM) {
      if (M <= 32) return launch_skinny<RB, 2, EPI, false, 0>(a, N, s);
      if (M <= 48) return launch_skinny<RB, 3, EPI, false, 0>(a, N, s);
      return launch_skinny<RB, 4, EPI, false, 0>(a, N, s);
    }
  } else {
    if (M <= 8) return launch_skinny<RB, 1, EPI, NRM, 1>(a, N, s);
    if (M <= 16) return launch_skinny<RB, 1, EPI, NRM, 2>(a, N, s);
    if constexpr (!NRM) {
      if (M <= 32) return launch_skinny<RB, 2, EPI, false, 2>(a, N, s);
      if (M <= 48) return launch_skinny<RB, 3, EPI, false, 2>(a, N, s);
      return launch_skinny<RB, 4, EPI, false, 2>(a, N, s);
    }
  }
  return hipErrorInvalidValue;
}

// ----------------------------------------------------------------------------
// wide GEMM: split-K partial sums of a batched decode's 9 to 64 rows and of token
// passes of 33 to 64 tokens on large weights
//
// A workgroup owns 128 weight rows (8 waves x 16) and one K split.  Every
// 128-wide K chunk of the activations (hi, and lo for the fp16 pair; all M
// tokens) is loaded once per workgroup into double-buffered LDS and read by
// all 8 waves as MFMA B fragments, so activation traffic is about the weight
// traffic instead of M/8 times it; each wave streams its own weight rows into
// registers, WP chunks ahead.  Waves own disjoint rows, so no reduction runs
// at the end: each writes its partial sums, and a reduction kernel applies
// the epilogue (part_store / part_resid / part_swiglu).

// LDS rows of 128 + 16 halves (288 bytes): the MFMA B-fragment reads (lane r
// reads row r, lanes 16 apart the next 16 bytes) are free of bank conflicts at
// that pitch; at 272 bytes every ds_read_b128 took 8 LDS cycles instead of 4.
// Three weight chunks in flight per wave: at 16 rows that fits 80 VGPRs, three
// workgroups per CU, and on the 7B shapes it beat four chunks by 1-5% (QKV at
// 16 rows 23.4 -> 22.1 us, O at 64 rows 15.1 -> 14.4 us; only O at 16 rows lost,
// 9.6 -> 9.9 us); six or eight chunks cost occupancy and were slower.
constexpr int WIDE_ROWS = 128, WIDE_WP = 3, WIDE_LDK = 128 + 16;

// weight fragments of one chunk of a wave's 16 rows from the fragment-ordered
// copy (1 KB of contiguous memory per MFMA step): wstrip = the strip's first
// block + lane * 8.  Measured against row-major loads (each lane 16 bytes of a
// different row) on the 7B shapes: at 64 rows gate|up 51.3 -> 48.8 us, QKV
// 32.6 -> 29.3 us, down 25.6 -> 24.2 us, O 13.2 -> 11.9 us; at 16 rows gate|up
// 38.4 -> 35.2 us, QKV 22.0 -> 20.1 us.
__device__ __forceinline__ void wide_wload_fo(uint4 (&w)[4], const f16* wstrip, int c) {
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = ld_stream(wstrip + ((size_t)c * 4 + i) * 512);
}

// one thread per 16 bytes of the fragment-ordered copy
__global__ __launch_bounds__(256) void k_frag_pack(const f16* __restrict__ W, int N, int K, f16* __restrict__ Wf) {
  const size_t o = (size_t)blockIdx.x * blockDim.x + threadIdx.x;  // 16-byte unit of Wf
  const size_t total = (size_t)N * K / 8;
  if (o >= total) return;
  const int l = (int)(o & 63);
  const size_t blk = o >> 6;  // (s * nch + c) * 4 + i
  const int i = (int)(blk & 3);
  const size_t sc = blk >> 2;
  const int nch = K >> 7;
  const int c = (int)(sc % nch);
  const size_t st = sc / nch;
  const size_t row = st * 16 + (l & 15), col = (size_t)c * 128 + 32 * i + 8 * (l >> 4);
  *(uint4*)(Wf + o * 8) = *(const uint4*)(W + row * K + col);
}

hipError_t frag_pack(const void* W, int N, int K, void* Wf, hipStream_t s) {
  if (N <= 0) return hipSuccess;
  if (N % 16 != 0 || K % 128 != 0) return hipErrorInvalidValue;
  const size_t units = (size_t)N * K / 8;
  hipLaunchKernelGGL(k_frag_pack, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, s, (const f16*)W, N, K,
                     (f16*)Wf);
  return hipGetLastError();
}

typedef unsigned u32x4v __attribute__((ext_vector_type(4)));
constexpr int WIDE_SC1 = 16;  // cache-policy bits of a buffer access: device scope (sc1)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t wide_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

// The reduction of one 128-column tile by the last of its splits to finish
// (EPI_STORE / EPI_RESID): every split's partial sums went out
// with device-scope stores, completed before the split counted itself in, so
// the last arrival reads them all (device-scope loads: the XCDs' L2s are not
// coherent with each other) and adds them in split order, the order the
// part_* reductions use.
struct WideEpi {
  unsigned* cnt;        // per-tile arrival counters, zero between launches (the last arrival resets its own)
  void* out;            // STORE: float [M][ldo]; SWIGLU: fp16 [M][ldo] (ldo = N / 2)
  void* olo;            // SWIGLU: rounding error of out (fp16) or NULL
  int ldo;
  float* h;             // RESID: residual [M][N] (+= the product)
  void* o16;            // RESID: fp16 pair of the new rows (o16, olo2) or NULL
  void* olo2;
  float* ss_out;        // RESID: sums of squares of the new rows per 128 columns, [M][N / 128], or NULL
  const float* ss_in;   // STORE / SWIGLU: the sums of squares of the unnormalised input rows, [M][K / 128], or NULL
  float eps;
};

// 1/rms of each of M input rows from their sums of squares per 128 columns, as
// row_rstd computes it (1 when ss is NULL), into rs; eight waves, no barrier.
__device__ __forceinline__ void wide_rstd(const float* ss, int M, int K, float eps, float* rs) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nss = K / 128;
  for (int m = wave; m < M; m += 8) {
    float t = 0.f;
    if (ss)
      for (int k = lane; k < nss; k += 64) t += ss[(size_t)m * nss + k];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
    if (lane == 0) rs[m] = ss ? 1.0f / sqrtf(t * (1.0f / (float)K) + eps) : 1.f;
  }
}

template <int EPI>
__device__ void wide_reduce(const WideEpi& e, __amdgpu_buffer_rsrc_t pr, int S, int M, int N, int K, int n0) {
  __shared__ float rs[64];
  const int tid = threadIdx.x;
  if constexpr (EPI != EPI_RESID) {
    wide_rstd(e.ss_in, M, K, e.eps, rs);
    __syncthreads();
  }
  auto sum4 = [&](int m, int n) {  // the S partials of 4 columns, added in split order
    float4 v = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < S; s0 += 4) {
      u32x4v q[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (s0 + j < S)
          q[j] = __builtin_amdgcn_raw_buffer_load_b128(pr, (uint32_t)((((size_t)(s0 + j) * M + m) * N + n) * 4), 0,
                                                       WIDE_SC1);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (s0 + j < S) {
          v.x += __uint_as_float(q[j][0]);
          v.y += __uint_as_float(q[j][1]);
          v.z += __uint_as_float(q[j][2]);
          v.w += __uint_as_float(q[j][3]);
        }
    }
    return v;
  };
  // 32 threads (half a wave) per row, 4 columns each
  for (int x = tid; x < ((M + 15) & ~15) * 32; x += blockDim.x) {
    const int m = x >> 5, n = n0 + 4 * (x & 31);
    const bool in = m < M;  // uniform over each half wave
    float4 v = {0.f, 0.f, 0.f, 0.f};
    if (in) v = sum4(m, n);
    if constexpr (EPI == EPI_STORE) {
      if (in) {
        const float sc = rs[m];
        *(float4*)((float*)e.out + (size_t)m * e.ldo + n) = float4{v.x * sc, v.y * sc, v.z * sc, v.w * sc};
      }
    } else {
      float q = 0.f;
      if (in) {
        float4* hp = (float4*)(e.h + (size_t)m * N + n);
        float4 hv = *hp;
        hv.x += v.x; hv.y += v.y; hv.z += v.z; hv.w += v.w;
        *hp = hv;
        if (e.o16) {
          const size_t o = (size_t)m * N + n;
          split16(hv.x, (f16*)e.o16, (f16*)e.olo2, o);
          split16(hv.y, (f16*)e.o16, (f16*)e.olo2, o + 1);
          split16(hv.z, (f16*)e.o16, (f16*)e.olo2, o + 2);
          split16(hv.w, (f16*)e.o16, (f16*)e.olo2, o + 3);
        }
        q = (hv.x * hv.x + hv.y * hv.y) + (hv.z * hv.z + hv.w * hv.w);
      }
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) q += __shfl_xor(q, o, 64);
      if (in && e.ss_out && (x & 31) == 0) e.ss_out[(size_t)m * (N / 128) + (n0 >> 7)] = q;
    }
  }
}

// The activation fragments of a K step are all requested before its first
// MFMA, so their LDS round trips overlap (one per MFMA otherwise); with 8 or
// more fragments a wave keeps two weight chunks in flight instead of three,
// which holds it at 120 VGPRs (four waves per SIMD).  On the 7B shapes at 64
// rows: gate|up 54.0 -> 50.8 us, QKV 32.7 -> 31.6 us, down 29.3 -> 25.5 us.
// The reduction fused into the last split (EPI_STORE / _RESID)
// measured 1-2 us faster per residual projection than GEMM + reduction kernel at
// 16 rows and 1-5 us slower at 64, where the O and down projections' 32 tiles
// then reduce on 32 CUs; the engine uses it up to 16 rows.  For SwiGLU with
// several splits it was slower at every row count (d = 2048, two splits, 16 rows:
// 13.4 against 9.9 us with k_part_swiglu).
template <int MB, int LO, int EPI>
__global__ __launch_bounds__(512) void k_gemm_wide(const f16* __restrict__ xhi, const f16* __restrict__ xlo,
                                                   const f16* __restrict__ W, int M, int K,
                                                   float* __restrict__ part, int N, WideEpi ep) {
  constexpr int NX = LO == 2 ? 2 : 1;               // activation arrays (hi, lo)
  constexpr int XCH = NX * MB * 16 * 16;             // 16-byte pieces of one staged chunk
  constexpr int XPT = (XCH + 511) / 512;             // pieces per thread
  constexpr int WP = MB * NX >= 6 ? 2 : WIDE_WP;     // weight chunks in flight
  extern __shared__ __attribute__((aligned(16))) f16 xs[];  // [2 stages][NX][MB*16][WIDE_LDK]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int n0 = blockIdx.x * WIDE_ROWS + wave * 16;
  const int nch = K >> 7, S = gridDim.y, sp = blockIdx.y;
  const int s0 = sp * nch / S, s1 = (sp + 1) * nch / S, n = s1 - s0;
  // the split's chunks in rotated order, by tile index / 8: the workgroups an XCD
  // runs at once (ids equal mod 8) start at different columns of their rows.
  // Measured on the 7B shapes: 1-5% faster at 16 rows (down 20.7 -> 19.6 us),
  // 0-1.5% at 64; rotating by the tile index itself was slower for gate|up.
  const int rot = n > 0 ? (int)((blockIdx.x >> 3) % (unsigned)n) : 0;
  auto chunk = [&](int t) { const int u = t + rot; return s0 + (u >= n ? u - n : u); };

  // W in fragment order: this wave's strip, lane's 16 bytes of each block
  const f16* wstrip = W + (size_t)(n0 / 16) * (K >> 7) * 2048 + lane * 8;
  uint4 wr[WP][4];
  // activation staging, up to 4 pieces of 16 bytes per thread (named registers:
  // an array here ends up on the stack).  Piece e = tid + 512 q: array
  // e / (MB*256), token row (e / 16) % (MB*16) (rows past M read row M-1: they
  // only feed token columns that are never stored), 16-byte column e % 16.
  static_assert(XPT <= 4, "at most 4 staging pieces per thread");
  uint4 x0 = {0u, 0u, 0u, 0u}, x1 = x0, x2 = x0, x3 = x0;
#define AMS_WIDE_XLOAD1(q, xq, c)                                                                  \
  do {                                                                                             \
    const int e_ = tid + 512 * (q);                                                                \
    if ((q) < XPT && (XCH % 512 == 0 || e_ < XCH)) {                                               \
      const int arr_ = e_ / (MB * 256), row_ = (e_ >> 4) % (MB * 16), col_ = e_ & 15;              \
      xq = *(const uint4*)((arr_ ? xlo : xhi) + (size_t)(row_ < M ? row_ : M - 1) * K + ((c) << 7) + col_ * 8); \
    }                                                                                              \
  } while (0)
#define AMS_WIDE_XSTORE1(q, xq, stage)                                                             \
  do {                                                                                             \
    const int e_ = tid + 512 * (q);                                                                \
    if ((q) < XPT && (XCH % 512 == 0 || e_ < XCH)) {                                               \
      const int arr_ = e_ / (MB * 256), row_ = (e_ >> 4) % (MB * 16), col_ = e_ & 15;              \
      *(uint4*)(xs + ((size_t)((stage) * NX + arr_) * MB * 16 + row_) * WIDE_LDK + col_ * 8) = xq; \
    }                                                                                              \
  } while (0)
#define AMS_WIDE_XLOAD(c) \
  do { AMS_WIDE_XLOAD1(0, x0, c); AMS_WIDE_XLOAD1(1, x1, c); AMS_WIDE_XLOAD1(2, x2, c); AMS_WIDE_XLOAD1(3, x3, c); } while (0)
#define AMS_WIDE_XSTORE(stage) \
  do { AMS_WIDE_XSTORE1(0, x0, stage); AMS_WIDE_XSTORE1(1, x1, stage); AMS_WIDE_XSTORE1(2, x2, stage); AMS_WIDE_XSTORE1(3, x3, stage); } while (0)

  f32x4 acc[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
  __shared__ float rs1[EPI == EPI_SWIGLU ? 64 : 1];
  if constexpr (EPI == EPI_SWIGLU) wide_rstd(ep.ss_in, M, K, ep.eps, rs1);

  // one K chunk t: its MFMAs from stage t & 1 and weights w, then staging chunk
  // t+1, the activation loads of chunk t+2 and the weight loads of chunk t+WP
  // (into w), each where that chunk exists.  The activation loads go out
  // before the weight loads: vmcnt retires in issue order, so staging chunk
  // t+2 next round waits only for loads older than the newest weight chunk.
  auto step = [&](int t, uint4 (&w)[4], bool st1, bool ld2, bool ldw) __attribute__((always_inline)) {
    const f16* xb = xs + (size_t)((t & 1) * NX) * MB * 16 * WIDE_LDK;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      half8 bf[NX][MB];
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int a = 0; a < NX; ++a)
          bf[a][mb] = *(const half8*)(xb + (size_t)(a * MB * 16 + mb * 16 + r) * WIDE_LDK + 32 * i + 8 * g);
      const half8 wf = as_half8(w[i]);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int a = 0; a < NX; ++a)
          acc[mb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf, bf[a][mb], acc[mb], 0, 0, 0);
    }
    if (st1) AMS_WIDE_XSTORE((t + 1) & 1);
    if (ld2) AMS_WIDE_XLOAD(chunk(t + 2));
    __builtin_amdgcn_sched_barrier(0);  // keep the issue order
    if (ldw) wide_wload_fo(w, wstrip, chunk(t + WP));
    __syncthreads();
  };
  int t = 0;
  if (n >= 2 * WP) {
    // Every chunk the prologue and the steps of this loop load exists, so
    // their loads are unconditional and issued in one order (a step's
    // activation loads, then its weight loads; the prologue X(c), W(c + WP - 2)
    // for c = 2 - WP .. 1): the loads in flight at the loop head are the same
    // from either edge, and the compiler's waits count them exactly instead of
    // draining them (with conditional loads each step waited for the weights
    // it had just requested).  Measured on the 7B decoder: 64-row decode 44.4
    // -> 44.0 ms per step, 16-row 56-token decode 223.0 -> 222.1 ms.
#pragma unroll
    for (int c = 2 - WP; c <= 1; ++c) {
      if (c >= 0) AMS_WIDE_XLOAD(chunk(c));
      __builtin_amdgcn_sched_barrier(0);
      wide_wload_fo(wr[c + WP - 2], wstrip, chunk(c + WP - 2));
      __builtin_amdgcn_sched_barrier(0);
      if (c == 0) AMS_WIDE_XSTORE(0);  // before the staging registers take chunk 1
    }
    __syncthreads();
    for (; t + 2 * WP <= n; t += WP) {
#pragma unroll
      for (int p = 0; p < WP; ++p) step(t + p, wr[p], true, true, true);
    }
  } else {
#pragma unroll
    for (int p = 0; p < WP; ++p)
      if (p < n) wide_wload_fo(wr[p], wstrip, chunk(p));
    AMS_WIDE_XLOAD(chunk(0));
    AMS_WIDE_XSTORE(0);
    if (n > 1) AMS_WIDE_XLOAD(chunk(1));
    __syncthreads();
  }
  // the remaining steps (fewer than 2 WP with the loop above)
  for (; t < n; t += WP) {
#pragma unroll
    for (int p = 0; p < WP; ++p)
      if (t + p < n) step(t + p, wr[p], t + p + 1 < n, t + p + 2 < n, t + p + WP < n);
  }

#undef AMS_WIDE_XLOAD1
#undef AMS_WIDE_XSTORE1
#undef AMS_WIDE_XLOAD
#undef AMS_WIDE_XSTORE

  // lane (r, g) holds rows n0 + 4g + i for token mb*16 + r
  if constexpr (EPI == EPI_PART) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int tok = mb * 16 + r;
      if (tok >= M) continue;
      float* dst = part + ((size_t)sp * M + tok) * N + n0 + 4 * g;
      *(float4*)dst = float4{acc[mb][0], acc[mb][1], acc[mb][2], acc[mb][3]};
    }
  } else if constexpr (EPI == EPI_SWIGLU) {  // one split: from registers
    // even waves hold gate rows, odd waves the up rows of the same 16 outputs: the up
    // values pass through the staging LDS, and the outputs leave without the partial
    // sums' trip through memory and without a second launch (7B gate|up, 16 rows: 37.6
    // us as four splits with their reduction, 33.6 as one split and k_part_swiglu, 32.0
    // so; 64 rows 52.2, 49.7 and 48.6)
    f32x4* up = (f32x4*)xs;  // [4 pairs][MB][64 lanes]; the last step's reads of xs are done (its barrier)
    if (wave & 1) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) up[((wave >> 1) * MB + mb) * 64 + lane] = acc[mb];
    }
    __syncthreads();
    if (wave & 1) return;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int tok = mb * 16 + r;
      if (tok >= M) continue;
      const f32x4 u4 = up[((wave >> 1) * MB + mb) * 64 + lane];
      const float sc = rs1[tok];
      const size_t o = (size_t)tok * ep.ldo + (n0 >> 1) + 4 * g;
      typedef _Float16 half4v __attribute__((ext_vector_type(4)));
      half4v hi, lo;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float y = silu(acc[mb][e] * sc) * (u4[e] * sc);
        hi[e] = sat16(y);
        lo[e] = sat16(y - (float)hi[e]);
      }
      *(half4v*)((f16*)ep.out + o) = hi;
      if (ep.olo) *(half4v*)((f16*)ep.olo + o) = lo;
    }
  } else {
    __shared__ int last;
    const __amdgpu_buffer_rsrc_t pr = wide_rsrc(part, (uint32_t)((size_t)S * M * N * 4));
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int tok = mb * 16 + r;
      if (tok >= M) continue;
      __builtin_amdgcn_raw_buffer_store_b128(u32x4v{__float_as_uint(acc[mb][0]), __float_as_uint(acc[mb][1]),
                                                    __float_as_uint(acc[mb][2]), __float_as_uint(acc[mb][3])},
                                             pr, (uint32_t)((((size_t)sp * M + tok) * N + n0 + 4 * g) * 4), 0,
                                             WIDE_SC1);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this thread's partial sums are stored
    __syncthreads();
    if (tid == 0) {
      unsigned* c = ep.cnt + blockIdx.x;
      const bool l = __hip_atomic_fetch_add(c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(S - 1);
      if (l) __hip_atomic_store(c, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // every split is in
      last = l;
    }
    __syncthreads();
    if (last) wide_reduce<EPI>(ep, pr, S, M, N, K, blockIdx.x * WIDE_ROWS);
  }
}

template <int MB, int LO, int EPI>
static hipError_t launch_wide(const f16* x, const f16* xlo, const f16* W, int M, int N, int K, int splits,
                              float* part, const WideEpi& ep, hipStream_t s) {
  const size_t lds = (size_t)2 * (LO == 2 ? 2 : 1) * MB * 16 * WIDE_LDK * sizeof(f16);
  hipLaunchKernelGGL((k_gemm_wide<MB, LO, EPI>), dim3(N / WIDE_ROWS, splits), dim3(512), lds, s, x, xlo, W, M, K,
                     part, N, ep);
  return hipGetLastError();
}

template <int EPI>
static hipError_t wide_epi(const void* u, const void* ulo, const void* W, int M, int N, int K, int splits, float* part,
                           const WideEpi& ep, hipStream_t s) {
  const f16 *x = (const f16*)u, *xl = (const f16*)ulo, *w = (const f16*)W;
  if (!ulo) {
    if constexpr (EPI == EPI_PART || EPI == EPI_SWIGLU) {
      if (M <= 16) return launch_wide<1, 0, EPI>(x, xl, w, M, N, K, splits, part, ep, s);
      if (M <= 32) return launch_wide<2, 0, EPI>(x, xl, w, M, N, K, splits, part, ep, s);
      if (M <= 48) return launch_wide<3, 0, EPI>(x, xl, w, M, N, K, splits, part, ep, s);
      return launch_wide<4, 0, EPI>(x, xl, w, M, N, K, splits, part, ep, s);
    }
    return hipErrorInvalidValue;  // the fused reductions serve the decode's pairs
  }
  if (M <= 16) return launch_wide<1, 2, EPI>(x, xl, w, M, N, K, splits, part, ep, s);
  if (M <= 32) return launch_wide<2, 2, EPI>(x, xl, w, M, N, K, splits, part, ep, s);
  if (M <= 48) return launch_wide<3, 2, EPI>(x, xl, w, M, N, K, splits, part, ep, s);
  return launch_wide<4, 2, EPI>(x, xl, w, M, N, K, splits, part, ep, s);
}

static bool wide_shape_ok(int M, int N, int K, int splits) {
  return M <= 64 && N % WIDE_ROWS == 0 && K % 128 == 0 && splits >= 1 && (K >> 7) >= splits;
}

hipError_t gemm_wide(const void* u, const void* ulo, const void* W, int M, int N, int K, int splits, float* part,
                     hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (!wide_shape_ok(M, N, K, splits)) return hipErrorInvalidValue;
  return wide_epi<EPI_PART>(u, ulo, W, M, N, K, splits, part, WideEpi{}, s);
}

hipError_t gemm_wide_reduce(int epi, const void* u, const void* ulo, const void* W, int M, int N, int K, int splits,
                            float* part, unsigned* counters, void* out, void* olo, int ldo, float* h, void* o16,
                            void* olo2, float* ss_out, const float* ss_in, float eps, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (!wide_shape_ok(M, N, K, splits) || !counters || !part) return hipErrorInvalidValue;
  if ((size_t)splits * M * N * 4 >= (size_t)1 << 31) return hipErrorInvalidValue;  // 32-bit buffer offsets
  WideEpi ep{counters, out, olo, ldo, h, o16, olo2, ss_out, ss_in, eps};
  switch (epi) {
    case EPI_STORE:
      if (!out || ldo < N) return hipErrorInvalidValue;
      return wide_epi<EPI_STORE>(u, ulo, W, M, N, K, splits, part, ep, s);
    case EPI_SWIGLU:
      if (!out || ldo < N / 2 || splits != 1) return hipErrorInvalidValue;
      return wide_epi<EPI_SWIGLU>(u, ulo, W, M, N, K, splits, part, ep, s);
    case EPI_RESID:
      if (!h || (olo2 && !o16)) return hipErrorInvalidValue;
      return wide_epi<EPI_RESID>(u, ulo, W, M, N, K, splits, part, ep, s);
    default:
      return hipErrorInvalidValue;
  }
}

// 1/rms of row m from the partial sums of squares k_part_resid left for it
// (ss[m][0..nss), added in a fixed order), shared with the whole block;
// 1 when ss is NULL.  Every thread of the block calls it.
__device__ float row_rstd(const float* __restrict__ ss, int nss, int m, float inv_n, float eps) {
  __shared__ float r;
  if (!ss) return 1.f;
  if (threadIdx.x < 64) {
    float t = 0.f;
    for (int k = threadIdx.x; k < nss; k += 64) t += ss[(size_t)m * nss + k];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
    if (threadIdx.x == 0) r = 1.0f / sqrtf(t * inv_n + eps);
  }
  __syncthreads();
  return r;
}

// out[m][n] = sum_s part[s][m][n] (splits added in order), times the row's
// 1/rms when ss is given (N a multiple of 256: a block lies in one row)
__global__ __launch_bounds__(256) void k_part_store(const float* __restrict__ part, int splits, size_t MN, int N,
                                                    const float* __restrict__ ss, int nss, float inv_n, float eps,
                                                    float* __restrict__ out) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  float v = 0.f;
  if (i < MN)
    for (int sp = 0; sp < splits; ++sp) v += part[sp * MN + i];
  // the row's scale after the partial loads are issued: both arrive in one round trip
  const float sc = row_rstd(ss, nss, (int)((size_t)blockIdx.x * blockDim.x / N), inv_n, eps);
  if (i < MN) out[i] = v * sc;
}

// a[m][c] = silu(gate) * up for the packed gate/up rows of output column c
// (16-row interleave), as an fp16 pair (out, olo); gate and up times the row's
// 1/rms when ss is given (N/2 a multiple of 256)
__global__ __launch_bounds__(256) void k_part_swiglu(const float* __restrict__ part, int splits, int M, int N,
                                                     const float* __restrict__ ss, int nss, float inv_n, float eps,
                                                     f16* __restrict__ out, f16* __restrict__ olo) {
  const int F = N / 2;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool in = i < (size_t)M * F;
  float gt = 0.f, up = 0.f;
  if (in) {
    const int m = (int)(i / F), c = (int)(i % F);
    const size_t gi = (size_t)m * N + (size_t)(c / GU_BLOCK) * 2 * GU_BLOCK + c % GU_BLOCK, MN = (size_t)M * N;
    for (int sp = 0; sp < splits; ++sp) {
      gt += part[sp * MN + gi];
      up += part[sp * MN + gi + GU_BLOCK];
    }
  }
  // the row's scale after the partial loads are issued: both arrive in one round trip
  const float sc = row_rstd(ss, nss, (int)((size_t)blockIdx.x * blockDim.x / F), inv_n, eps);
  if (in) split16(silu(gt * sc) * (up * sc), out, olo, i);
}

hipError_t part_store(const float* part, int splits, int M, int N, float* out, hipStream_t s, const float* ss,
                      int d, float eps) {
  if (M <= 0) return hipSuccess;
  if (ss && (N % 256 != 0 || d <= 0 || d % 256 != 0)) return hipErrorInvalidValue;
  const size_t MN = (size_t)M * N;
  hipLaunchKernelGGL(k_part_store, dim3((unsigned)((MN + 255) / 256)), dim3(256), 0, s, part, splits, MN, N, ss,
                     d / 128, ss ? 1.0f / (float)d : 0.f, eps, out);
  return hipGetLastError();
}

hipError_t part_swiglu(const float* part, int splits, int M, int N, void* out, void* olo, hipStream_t s,
                       const float* ss, int d, float eps) {
  if (M <= 0) return hipSuccess;
  if (N % (2 * GU_BLOCK) != 0) return hipErrorInvalidValue;
  if (ss && ((N / 2) % 256 != 0 || d <= 0 || d % 256 != 0)) return hipErrorInvalidValue;
  const size_t MF = (size_t)M * (N / 2);
  hipLaunchKernelGGL(k_part_swiglu, dim3((unsigned)((MF + 255) / 256)), dim3(256), 0, s, part, splits, M, N, ss,
                     d / 128, ss ? 1.0f / (float)d : 0.f, eps, (f16*)out, (f16*)olo);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------
// split-K decode GEMV: partial sums of `splits` K ranges, then a reduction

hipError_t gemm_part(const void* u, const void* ulo, const void* W, int M, int N, int K, int splits, float* part,
                     hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (M > 64 || splits < 1 || (K >> 7) < splits) return hipErrorInvalidValue;
  const SkinnyArgs a{(const f16*)u, (const f16*)ulo, 0.f, (const f16*)W, M, K, part, N, nullptr, nullptr};
  if (!ulo) {
    if (M <= 16) return launch_skinny<1, 1, EPI_PART, false, 0>(a, N, s, splits);
    if (M <= 32) return launch_skinny<1, 2, EPI_PART, false, 0>(a, N, s, splits);
    if (M <= 48) return launch_skinny<1, 3, EPI_PART, false, 0>(a, N, s, splits);
    return launch_skinny<1, 4, EPI_PART, false, 0>(a, N, s, splits);
  }
  if (M <= 8) return launch_skinny<1, 1, EPI_PART, false, 1>(a, N, s, splits);
  if (M <= 16) return launch_skinny<1, 1, EPI_PART, false, 2>(a, N, s, splits);
  if (M <= 32) return launch_skinny<1, 2, EPI_PART, false, 2>(a, N, s, splits);
  if (M <= 48) return launch_skinny<1, 3, EPI_PART, false, 2>(a, N, s, splits);
  return launch_skinny<1, 4, EPI_PART, false, 2>(a, N, s, splits);
}

// h[m][n] += sum_s part[s][m][n] (splits in order), and the fp16 pair of the
// updated row when o16 is non-NULL; with ss, each block (256 columns of one
// row: N a multiple of 256) also leaves the sums of squares of its new values
// per 128 columns at ss[2 blockIdx ..], i.e. ss[m][n / 128], for the next
// projection's RMSNorm
__global__ __launch_bounds__(256) void k_part_resid(const float* __restrict__ part, int splits, int M, int N,
                                                    float* __restrict__ h, f16* __restrict__ o16,
                                                    f16* __restrict__ olo, float* __restrict__ ss) {
  __shared__ float wsq[4];
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t MN = (size_t)M * N;
  float hn = 0.f;
  if (i < MN) {
    float v = 0.f;
    for (int sp = 0; sp < splits; ++sp) v += part[sp * MN + i];
    hn = h[i] + v;
    h[i] = hn;
    if (o16) split16(hn, o16, olo, i);
  }
  if (!ss) return;
  float q = hn * hn;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) q += __shfl_xor(q, o, 64);
  if ((threadIdx.x & 63) == 0) wsq[threadIdx.x >> 6] = q;
  __syncthreads();
  if (threadIdx.x < 2) ss[2 * blockIdx.x + threadIdx.x] = wsq[2 * threadIdx.x] + wsq[2 * threadIdx.x + 1];
}

hipError_t part_resid(const float* part, int splits, int M, int N, float* h, void* o16, void* olo, hipStream_t s,
                      float* ss) {
  if (M <= 0) return hipSuccess;
  if ((olo && !o16) || (ss && N % 256 != 0)) return hipErrorInvalidValue;
  const size_t MN = (size_t)M * N;
  hipLaunchKernelGGL(k_part_resid, dim3((unsigned)((MN + 255) / 256)), dim3(256), 0, s, part, splits, M, N, h,
                     (f16*)o16, (f16*)olo, ss);
  return hipGetLastError();
}

template <int EPI>
static hipError_t gemm_epi(int ct, const void* u, const void* W, int M, int N, int K, void* out, int ldo,
                           hipStream_t s, const void* ulo, void* o16, void* olo) {
  const bool pair = ulo || o16 || olo;
  if (pair) {  // the fp16-pair forms belong to the decode GEMV only
    if (ct != DT_F16 || M > 64) return hipErrorInvalidValue;
    if (o16 && EPI != EPI_RESID) return hipErrorInvalidValue;
    if (olo && EPI == EPI_STORE) return hipErrorInvalidValue;
    if (olo && EPI == EPI_RESID && !o16) return hipErrorInvalidValue;
  }
  if (ct == DT_F32) return gemm_f32(EPI, (const float*)u, (const float*)W, M, N, K, (float*)out, ldo, s);
  if (M <= 64) {
    const SkinnyArgs a{(const f16*)u, (const f16*)ulo, 0.f, (const f16*)W, M, K, out, ldo, (f16*)o16, (f16*)olo};
    return skinny_dispatch<EPI, false>(a, N, s);
  }
  return hipErrorInvalidValue;  // longer token passes: gemm_tokens
}

hipError_t gemm(int ct, int epi, const void* u, const void* W, int M, int N, int K, void* out, int ldo,
                hipStream_t s, const void* ulo, void* o16, void* olo) {
  if (M <= 0) return hipSuccess;
  switch (epi) {
    case EPI_STORE: return gemm_epi<EPI_STORE>(ct, u, W, M, N, K, out, ldo, s, ulo, o16, olo);
    case EPI_RESID: return gemm_epi<EPI_RESID>(ct, u, W, M, N, K, out, ldo, s, ulo, o16, olo);
    default: return gemm_epi<EPI_SWIGLU>(ct, u, W, M, N, K, out, ldo, s, ulo, o16, olo);
  }
}

// Token passes: FRAG.  From row-major weights a wave's loads were 64-byte pieces of 16
// rows (7B, 16 tokens: QKV 31.2 -> 22.8 us, gate|up 47.2 -> 39.3, O 12.1 -> 9.1, down
// 27.2 -> 19.9; same sums).
template <int EPI> static hipError_t tokens_short(const SkinnyArgs& a, int N, hipStream_t s) {
  constexpr int RB = EPI == EPI_SWIGLU ? 2 : 1;
  if (a.M <= 16) return launch_skinny<RB, 1, EPI, false, 0, true>(a, N, s);
  if (a.M <= 32) return launch_skinny<RB, 2, EPI, false, 0, true>(a, N, s);
  if (a.M <= 48) return launch_skinny<RB, 3, EPI, false, 0, true>(a, N, s);
  return launch_skinny<RB, 4, EPI, false, 0, true>(a, N, s);
}

hipError_t gemm_tokens_short(int epi, const void* u, const void* Wf, int M, int N, int K, void* out, int ldo,
                             hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (M > 64 || N % (epi == EPI_SWIGLU ? 32 : 16) != 0 || K % 128 != 0) return hipErrorInvalidValue;
  const SkinnyArgs a{(const f16*)u, nullptr, 0.f, (const f16*)Wf, M, K, out, ldo, nullptr, nullptr};
  switch (epi) {
    case EPI_STORE: return tokens_short<EPI_STORE>(a, N, s);
    case EPI_RESID: return tokens_short<EPI_RESID>(a, N, s);
    case EPI_SWIGLU: return tokens_short<EPI_SWIGLU>(a, N, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t gemv_rmsnorm(int ct, int epi, const void* hhi, float eps, const void* W, int M, int N, int K, void* out,
                        int ldo, hipStream_t s, const void* hlo, void* o16, void* olo) {
  if (M <= 0) return hipSuccess;
  if (ct != DT_F16 || M > 16) return hipErrorInvalidValue;
  if (o16 && epi != EPI_RESID) return hipErrorInvalidValue;
  if (olo && (epi == EPI_STORE || (epi == EPI_RESID && !o16))) return hipErrorInvalidValue;
  const SkinnyArgs a{(const f16*)hhi, (const f16*)hlo, eps, (const f16*)W, M, K, out, ldo, (f16*)o16, (f16*)olo};
  switch (epi) {
    case EPI_STORE: return skinny_dispatch<EPI_STORE, true>(a, N, s);
    case EPI_RESID: return skinny_dispatch<EPI_RESID, true>(a, N, s);
    default: return skinny_dispatch<EPI_SWIGLU, true>(a, N, s);
  }
}

}  // namespace ams
