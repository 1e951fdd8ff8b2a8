// fp16 projections of token passes (more than 64 tokens: prefix builds,
// observation extensions, flow chunks): y = u W^T with u row-major and W in MFMA
// fragment order (frag_pack), fp32 accumulation in K order on every tile shape, so
// that the shape a pass's token count picks does not show in its results; fused epilogues.
//
// Both kernels move their tiles from global memory straight into LDS
// (global_load_lds_dwordx4: a wave instruction fills 1 KB, lane i the i-th 16
// bytes).  A weight block is one MFMA fragment, 1 KB of contiguous memory that
// lands in LDS as the fragment reads want it; rows of u go to swizzled slots, so
// that the 16-byte fragment reads of either operand meet every LDS bank once.
// The weights are the A operand of the MFMA: a lane ends up with 4 consecutive
// outputs of one token, which it stores as one 16-byte (fp32) or 8-byte (fp16) word.
//
//  * k_tok_pp: 256 x 256 tiles, one workgroup of 8 waves per CU, for passes with
//    enough of them.  Bound by the MFMA rate.
//  * k_tok_pipe: smaller tiles with one to five K steps of loads in flight, for
//    passes whose 256 x 256 tiles would leave CUs idle.  Bound by the latency and
//    rate of the operand loads.
#include <atomic>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace ams {

typedef __attribute__((address_space(3))) void* lds_ptr;
typedef _Float16 half4v __attribute__((ext_vector_type(4)));

template <int N> __device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// Tile of a workgroup.  Workgroups are dispatched round-robin over the 8 XCDs:
// XCD x (ids = x mod 8) takes a contiguous range of a tile sequence that walks
// groups of 8 token tiles down each weight tile, so tiles that share operands
// run close together on one XCD's L2.
template <int BM, int BN> __device__ __forceinline__ void tok_tile(int M, int N, int& m0, int& n0) {
  const int tm_n = (M + BM - 1) / BM, tn_n = N / BN, T = tm_n * tn_n;
  const int L = blockIdx.x, xcd = L & 7, per = T >> 3, rem = T & 7;
  const int Lx = xcd * per + (xcd < rem ? xcd : rem) + (L >> 3);
  const int grp = Lx / (8 * tn_n), first_m = grp * 8;
  const int gm = tm_n - first_m < 8 ? tm_n - first_m : 8;
  const int in_grp = Lx - grp * 8 * tn_n;
  m0 = (first_m + in_grp % gm) * BM;
  n0 = (in_grp / gm) * BN;
}

// Epilogue of one token's blocks: acc[j] = outputs col(j) + 4g .. + 3 of token
// tok, col(j) the first weight row of the wave's j-th 16-row strip.
template <int EPI, int NJ, typename Col>
__device__ __forceinline__ void tok_epilogue(const f32x4 (&acc)[NJ], Col col, int g, int tok, int M, int sp,
                                             void* __restrict__ out, int ldo) {
  if constexpr (EPI == EPI_SWIGLU) {  // strips 2p (gate) and 2p + 1 (up) of the packed interleave
#pragma unroll
    for (int p = 0; p < NJ / 2; ++p) {
      half4v y;
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = sat16(silu(acc[2 * p][e]) * acc[2 * p + 1][e]);
      *(half4v*)((f16*)out + (size_t)tok * ldo + (col(2 * p) >> 1) + 4 * g) = y;
    }
  } else {
    float* row = (float*)out + ((size_t)(EPI == EPI_PART ? sp * M : 0) + tok) * ldo + 4 * g;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      f32x4* p = (f32x4*)(row + col(j));
      if constexpr (EPI == EPI_RESID) *p += acc[j];
      else *p = acc[j];
    }
  }
}

// ----------------------------------------------------------------------------
// 256 x 256 tiles, two groups of four waves half a K step apart.
//
// Waves 0-3 (one per SIMD) own tokens 0..127 of the tile, waves 4-7 (the other
// wave of each SIMD) tokens 128..255; a wave covers 4 strips of weight rows.  K
// goes in steps of 32 through four LDS slots.  Each step has two phases with a
// workgroup barrier after each: read the step's 12 fragments (and request the
// slot three steps ahead), then its 32 MFMAs.  The second group runs one phase
// behind, so on every SIMD one wave's MFMAs cover the other's LDS reads and
// waits; with all eight waves in step (every fragment requested in use order, one
// barrier per K step of 64) the matrix cores stood idle at each barrier.
// Measured at 19,200 tokens of the 7B shapes: QKV 1,883 -> 1,637 us, gate|up
// 2,998 -> 2,691 us, down 1,623 -> 1,457 us (1.18-1.29 PFLOP/s); at 1,024 tokens
// QKV 102.5 -> 99 us.  Weights in fragment order are part of it: row-major weights
// in 64-byte pieces ran 1,800 us at the QKV shape.
//
// A slot is refilled by the loads issued in the read phase one step after its
// last reader's: group 2's read phase of a step ends (its fragments waited for)
// before the barrier that opens group 1's read phase of the next.  A step's loads
// are waited for by the waves that issued them before the barrier that precedes
// group 1's read phase of that step; loads of the two later steps stay in flight.
constexpr int PP_SLOTS = 4, PP_LPW = 4, PP_SLOT = 32 * 1024;

template <int EPI, int DH>  // DH: head_dim (EPI_QKV)
__global__ __launch_bounds__(512) void k_tok_pp(const f16* __restrict__ u, const f16* __restrict__ W, int M, int N,
                                                int K, void* __restrict__ out, int ldo, KvEpi kv) {
  constexpr int NI = 8, NJ = 4;
  extern __shared__ __attribute__((aligned(16))) unsigned char tsm[];  // [slot][16 token | 16 weight blocks of 1 KB]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4, wm = wave >> 2, wn = wave & 3;
  int m0, n0;
  tok_tile<256, 256>(M, N, m0, n0);
  const int alast = M - 1 - m0;  // last valid token row of the tile
  const int KT = K / 64, sp = blockIdx.y, S = gridDim.y;
  const int kt0 = sp * KT / S, KS = 2 * ((sp + 1) * KT / S - kt0);  // steps of 32 of this split
  // the wave's strips; heads of 128 keep a rotation pair (strips 4 apart) in one lane
  auto strip = [&](int j) { return EPI == EPI_QKV && DH == 128 ? wn + 4 * j : wn * NJ + j; };

  // this wave's 4 of a slot's 32 blocks: token block b holds rows 16b.. (16 rows x
  // 64 bytes; 16-byte chunk c of row i sits at slot c ^ (i / 4) of the row)
  const f16* src[PP_LPW];
#pragma unroll
  for (int q = 0; q < PP_LPW; ++q) {
    const int blk = wave * PP_LPW + q;
    if (blk < 16) {
      int row = lane >> 2;
      const int c = (lane & 3) ^ (row >> 2);
      row += blk * 16;
      if (row > alast) row = alast;  // feeds outputs that are never stored
      src[q] = u + (size_t)(m0 + row) * K + kt0 * 64 + c * 8;
    } else {
      src[q] = W + ((size_t)(n0 / 16 + blk - 16) * (K / 32) + 2 * kt0) * 512 + lane * 8;
    }
  }
  auto dma = [&](int s) __attribute__((always_inline)) {
    unsigned char* st = tsm + (s % PP_SLOTS) * PP_SLOT;
#pragma unroll
    for (int q = 0; q < PP_LPW; ++q) {
      const int blk = wave * PP_LPW + q;
      __builtin_amdgcn_global_load_lds((const void*)(src[q] + (size_t)s * (blk < 16 ? 32 : 512)),
                                       (lds_ptr)(st + blk * 1024), 16, 0, 0);
    }
  };
  const int toff = (r * 4 + (g ^ (r >> 2))) * 16;  // this lane's chunk of a token block
  f32x4 acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  half8 tf[NI], wf[NJ];
  auto read = [&](int s) __attribute__((always_inline)) {
    const unsigned char* cur = tsm + (s % PP_SLOTS) * PP_SLOT;
#pragma unroll
    for (int i = 0; i < NI; ++i) tf[i] = *(const half8*)(cur + (wm * NI + i) * 1024 + toff);
#pragma unroll
    for (int j = 0; j < NJ; ++j) wf[j] = *(const half8*)(cur + (16 + strip(j)) * 1024 + lane * 16);
    if (s + PP_SLOTS - 1 < KS) dma(s + PP_SLOTS - 1);
  };
  // this wave's loads of step s have landed
  auto landed = [&](int s) __attribute__((always_inline)) {
    if (s + PP_SLOTS - 2 < KS) wait_vm<(PP_SLOTS - 2) * PP_LPW>();
    else wait_vm<0>();
  };
  auto barrier = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int s = 0; s < PP_SLOTS - 1; ++s)
    if (s < KS) dma(s);
  landed(0);
  barrier();
  if (wave >= 4) barrier();  // the second group starts one phase later
  for (int s = 0; s < KS; ++s) {
    read(s);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (wave >= 4 && s + 1 < KS) landed(s + 1);
    barrier();
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int i = 0; i < NI; ++i)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[j], tf[i], acc[i][j], 0, 0, 0);
    if (wave < 4 && s + 1 < KS) landed(s + 1);
    barrier();
  }
  if (wave < 4) barrier();

#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int tok = m0 + wm * 128 + i * 16 + r;
    if (tok >= M) continue;
    auto col = [&](int j) { return n0 + 16 * strip(j); };
    if constexpr (EPI == EPI_QKV) {
      // q columns stored fp32 for the attention; k (rotated at the token's position,
      // rotate-half) and v written fp16 to the token's pool slot, as k_kv_append_tab
      // writes them (d is a multiple of 256, so a tile lies in one of q, k, v)
      if (n0 < kv.d) {
        tok_epilogue<EPI_STORE>(acc[i], col, g, tok, M, sp, out, ldo);
        continue;
      }
      constexpr int HALF = DH / 2;
      const bool isk = n0 < 2 * kv.d;
      f16* dst = (f16*)(isk ? kv.k : kv.v) + (size_t)kv.tok_base[tok];
      const int c0 = n0 - (isk ? kv.d : 2 * kv.d);
      if (isk) {
        const int p = kv.tok_pos[tok];
        // strips j and j + DP hold dims dd and dd + HALF of a head (128: strips 4 apart,
        // held as neighbours; 64: strips 2 apart of the wave's own head)
        constexpr int DP = DH == 128 ? 1 : 2;
#pragma unroll
        for (int x = 0; x < NJ / 2; ++x) {
          const int j = DH == 128 ? 2 * x : x;
          const int cc = c0 + 16 * strip(j) + 4 * g, h = cc / DH, dd = cc % DH;
          const float4 r0 = *(const float4*)(kv.rope + (size_t)p * HALF + dd);
          const float4 r1 = *(const float4*)(kv.rope + (size_t)p * HALF + dd + 2);
          const float cx[4] = {r0.x, r0.z, r1.x, r1.z}, cy[4] = {r0.y, r0.w, r1.y, r1.w};
          half4v lo, hi;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float l, u;
            rope_pair(acc[i][j][e], acc[i][j + DP][e], cx[e], cy[e], l, u);
            lo[e] = sat16(l);
            hi[e] = sat16(u);
          }
          f16* kd = dst + (size_t)h * KV_PAGE * DH + dd;
          *(half4v*)kd = lo;
          *(half4v*)(kd + HALF) = hi;
        }
      } else {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int cc = c0 + 16 * strip(j) + 4 * g, h = cc / DH, dd = cc % DH;
          *(half4v*)(dst + (size_t)h * KV_PAGE * DH + dd) =
              half4v{sat16(acc[i][j][0]), sat16(acc[i][j][1]), sat16(acc[i][j][2]), sat16(acc[i][j][3])};
        }
      }
    } else {
      tok_epilogue<EPI>(acc[i], col, g, tok, M, sp, out, ldo);
    }
  }
}

// ----------------------------------------------------------------------------
// BM tokens x BN weight rows, WM x WN waves, K steps of 64 through NST LDS stages
// with one barrier per step: a wave waits for its own loads of the step (issued
// NST - 1 steps earlier), the barrier makes every wave's visible and says that the
// stage of the step before is read out, and the loads NST - 1 steps ahead go into
// it.  With one step prefetched into registers (128 x 128 tiles) a step cost a
// whole memory round trip, 1.2 us, whatever its size.  Measured on the 7B
// shapes: 128 tokens QKV 82 -> 33 us, gate|up 82 -> 49 us; 288 tokens QKV 73 -> 51;
// 600 tokens QKV 89 -> 72 us, down (six ranges, without their reduction) 100 -> 73.
// The 128 x 64 tile and the two 128 x 128 workgroups of a CU have eight waves of 32
// x 32 and 64 x 32: four left a SIMD one wave, which waited for the same stage as the
// others (QKV of the 7B width at 128 tokens 34.0 -> 31.9 us, 30.9 -> 28.5 at 72; 288
// tokens of two 128 x 128 workgroups 60.9 -> 60.0).
// SEG (a residual projection whose K ranges one workgroup adds): each range's sums
// start from zero and are added in order, as the reduction of partial sums adds them.
template <int EPI, int BM, int BN, int WM, int WN, int NST, bool SEG>
__global__ __launch_bounds__(64 * WM * WN) void k_tok_pipe(const f16* __restrict__ u, const f16* __restrict__ W, int M,
                                                           int N, int K, void* __restrict__ out, int ldo, int segs) {
  constexpr int NW = WM * WN, TM = BM / WM, TN = BN / WN, NI = TM / 16, NJ = TN / 16;
  constexpr int AB = BM / 8, BB = BN / 8, LPW = (AB + BB) / NW;  // 1 KB blocks of a stage, loads per wave
  constexpr int STAGE = (AB + BB) * 1024;
  static_assert((AB + BB) % NW == 0, "every wave issues as many loads per stage");
  static_assert(EPI != EPI_SWIGLU || NJ % 2 == 0, "gate and up strips come in pairs");
  extern __shared__ __attribute__((aligned(16))) unsigned char tsm[];  // [stage][AB token | BB weight blocks]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4, wm = wave / WN, wn = wave % WN;
  int m0, n0;
  tok_tile<BM, BN>(M, N, m0, n0);
  const int alast = M - 1 - m0;
  const int KTa = K / 64, sp = blockIdx.y, S = gridDim.y;
  const int kt0 = sp * KTa / S, KT = (sp + 1) * KTa / S - kt0;

  // token block b: rows 8b.. of 128 bytes, chunk c of row i at slot c ^ (i & 7);
  // weight block b: step b & 1 of strip b / 2
  const f16* src[LPW];
#pragma unroll
  for (int q = 0; q < LPW; ++q) {
    const int blk = wave * LPW + q;
    if (blk < AB) {
      int row = blk * 8 + (lane >> 3);
      const int c = (lane & 7) ^ (row & 7);
      if (row > alast) row = alast;  // feeds outputs that are never stored
      src[q] = u + (size_t)(m0 + row) * K + (size_t)kt0 * 64 + c * 8;
    } else {
      const int b = blk - AB;
      src[q] = W + ((size_t)(n0 / 16 + b / 2) * (K / 32) + 2 * kt0 + (b & 1)) * 512 + lane * 8;
    }
  }
  auto dma = [&](int t) __attribute__((always_inline)) {
    unsigned char* st = tsm + (t % NST) * STAGE;
#pragma unroll
    for (int q = 0; q < LPW; ++q) {
      const int blk = wave * LPW + q;
      __builtin_amdgcn_global_load_lds((const void*)(src[q] + (size_t)t * (blk < AB ? 64 : 1024)),
                                       (lds_ptr)(st + blk * 1024), 16, 0, 0);
    }
  };
  f32x4 acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 tot[SEG ? NI : 1][SEG ? NJ : 1];
  int seg = 1, seg_end = KT / segs;  // the range this K step lies in, and its end
  if constexpr (SEG)
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) tot[i][j] = acc[i][j];
#pragma unroll
  for (int t = 0; t < NST - 1; ++t)
    if (t < KT) dma(t);
  for (int t = 0; t < KT; ++t) {
    if (t + NST - 2 < KT) wait_vm<(NST - 2) * LPW>();
    else wait_vm<0>();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the stage that is refilled next is read out
    __builtin_amdgcn_s_barrier();
    if (t + NST - 1 < KT) dma(t + NST - 1);
    const unsigned char* cur = tsm + (t % NST) * STAGE;
    const unsigned char* Tb = cur + (wm * TM + r) * 128;
    const unsigned char* Wb = cur + AB * 1024 + wn * NJ * 2048 + lane * 16;
    half8 tf[2][NI], wf[2][NJ];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
#pragma unroll
      for (int i = 0; i < NI; ++i) tf[k][i] = *(const half8*)(Tb + i * 2048 + (((4 * k + g) ^ (r & 7)) << 4));
#pragma unroll
      for (int j = 0; j < NJ; ++j) wf[k][j] = *(const half8*)(Wb + (2 * j + k) * 1024);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < NI; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[k][j], tf[k][i], acc[i][j], 0, 0, 0);
    if constexpr (SEG) {
      if (t + 1 == seg_end) {
        seg_end = ++seg * KT / segs;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            tot[i][j] += acc[i][j];
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
      }
    }
  }
  auto& y = [&]() -> f32x4(&)[NI][NJ] {
    if constexpr (SEG) return tot;
    else return acc;
  }();
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int tok = m0 + wm * TM + i * 16 + r;
    if (tok < M)
      tok_epilogue<EPI>(y[i], [&](int j) { return n0 + wn * TN + 16 * j; }, g, tok, M, sp, out, ldo);
  }
}

// ----------------------------------------------------------------------------

// Allows `kernel` `bytes` of dynamic LDS on the current device, once per device (done: a bit each).
static hipError_t lds_limit(std::atomic<uint64_t>& done, const void* kernel, int bytes) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev < 64 ? (uint64_t)1 << dev : 0;
  if (done.load(std::memory_order_relaxed) & bit) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_relaxed);
  return e;
}

template <int EPI, int DH = 128>
static hipError_t launch_pp(const f16* u, const f16* W, int M, int N, int K, void* out, int ldo, int splits,
                            const KvEpi& kv, hipStream_t s) {
  static std::atomic<uint64_t> done{0};
  const hipError_t lim = lds_limit(done, (const void*)k_tok_pp<EPI, DH>, PP_SLOTS * PP_SLOT);
  if (lim != hipSuccess) return lim;
  hipLaunchKernelGGL((k_tok_pp<EPI, DH>), dim3((N / 256) * ((M + 255) / 256), splits), dim3(512), PP_SLOTS * PP_SLOT, s,
                     u, W, M, N, K, out, ldo, kv);
  return hipGetLastError();
}

template <int EPI, int BM, int BN, int WM, int WN, int NST, bool SEG>
static hipError_t launch_pipe(const f16* u, const f16* W, int M, int N, int K, void* out, int ldo, int splits,
                              int segs, hipStream_t s) {
  constexpr int LDS = NST * (BM + BN) * 128;
  static std::atomic<uint64_t> done{0};
  const hipError_t lim = lds_limit(done, (const void*)k_tok_pipe<EPI, BM, BN, WM, WN, NST, SEG>, LDS);
  if (lim != hipSuccess) return lim;
  hipLaunchKernelGGL((k_tok_pipe<EPI, BM, BN, WM, WN, NST, SEG>), dim3((N / BN) * ((M + BM - 1) / BM), splits),
                     dim3(64 * WM * WN), LDS, s, u, W, M, N, K, out, ldo, segs);
  return hipGetLastError();
}

template <int EPI, bool SEG = false>
static hipError_t tok_epi(int tile, const f16* u, const f16* W, int M, int N, int K, void* out, int ldo, int splits,
                          int segs, hipStream_t s) {
  switch (tile) {
    case TT_256x256:
      if constexpr (!SEG) return launch_pp<EPI>(u, W, M, N, K, out, ldo, splits, KvEpi{}, s);
      return hipErrorInvalidValue;
    case TT_128x256: return launch_pipe<EPI, 128, 256, 2, 4, 3, SEG>(u, W, M, N, K, out, ldo, splits, segs, s);
    case TT_256x128: return launch_pipe<EPI, 256, 128, 4, 2, 3, SEG>(u, W, M, N, K, out, ldo, splits, segs, s);
    case TT_128x128x2: return launch_pipe<EPI, 128, 128, 2, 4, 2, SEG>(u, W, M, N, K, out, ldo, splits, segs, s);
    case TT_128x128: return launch_pipe<EPI, 128, 128, 4, 2, 4, SEG>(u, W, M, N, K, out, ldo, splits, segs, s);
    case TT_64x128: return launch_pipe<EPI, 64, 128, 1, 4, 3, SEG>(u, W, M, N, K, out, ldo, splits, segs, s);
    case TT_64x256: return launch_pipe<EPI, 64, 256, 1, 8, 4, SEG>(u, W, M, N, K, out, ldo, splits, segs, s);
    case TT_128x64: return launch_pipe<EPI, 128, 64, 4, 2, 6, SEG>(u, W, M, N, K, out, ldo, splits, segs, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t gemm_tokens_tile(int tile, int epi, const void* u, const void* Wf, int M, int N, int K, void* out, int ldo,
                            int splits, hipStream_t s, int segs) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (tile < 0 || tile >= TT_COUNT || N % TOK_TILES[tile].bn != 0 || K % 64 != 0 || splits < 1 || splits > K / 64 ||
      (splits > 1 && epi != EPI_PART) || segs < 1 || segs > K / 64 || (segs > 1 && epi != EPI_RESID))
    return hipErrorInvalidValue;
  const f16 *x = (const f16*)u, *w = (const f16*)Wf;
  switch (epi) {
    case EPI_STORE: return tok_epi<EPI_STORE>(tile, x, w, M, N, K, out, ldo, 1, 1, s);
    case EPI_RESID:
      if (segs > 1) return tok_epi<EPI_RESID, true>(tile, x, w, M, N, K, out, ldo, 1, segs, s);
      return tok_epi<EPI_RESID>(tile, x, w, M, N, K, out, ldo, 1, 1, s);
    case EPI_SWIGLU: return tok_epi<EPI_SWIGLU>(tile, x, w, M, N, K, out, ldo, 1, 1, s);
    case EPI_PART: return tok_epi<EPI_PART>(tile, x, w, M, N, K, out, N, splits, 1, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t gemm_tokens(int epi, const void* u, const void* Wf, int M, int N, int K, void* out, int ldo,
                       hipStream_t s) {
  const TokPlan p = tok_plan(M, N, K, 1, true);
  hipError_t e = gemm_tokens_tile(p.tile, epi, u, Wf, M, p.main_n, K, out, ldo, 1, s);
  if (e != hipSuccess || p.rest_tile < 0) return e;
  // the weight rows past main_n (output columns main_n / 2 on for SwiGLU)
  void* o2 = epi == EPI_SWIGLU ? (void*)((f16*)out + p.main_n / 2) : (void*)((float*)out + p.main_n);
  return gemm_tokens_tile(p.rest_tile, epi, u, (const f16*)Wf + (size_t)p.main_n * K, M, N - p.main_n, K, o2, ldo, 1,
                          s);
}

bool gemm_qkv_fusable(int M, int N, int dh, int d) {
  if (M <= 64 || (dh != 64 && dh != 128) || d % 256 != 0 || N != 3 * d) return false;
  return (size_t)(N / 256) * ((M + 255) / 256) > 256 && tok_plan(M, N, d, 1, false).tile == TT_256x256;
}

hipError_t gemm_qkv_kv(const void* u, const void* Wf, int M, int K, float* qkv, const KvEpi& kv, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if ((kv.dh != 64 && kv.dh != 128) || kv.d <= 0 || kv.d % 256 != 0 || K % 64 != 0 || !kv.tok_base || !kv.tok_pos ||
      !kv.k || !kv.v || !kv.rope)
    return hipErrorInvalidValue;
  const f16 *x = (const f16*)u, *w = (const f16*)Wf;
  if (kv.dh == 128) return launch_pp<EPI_QKV, 128>(x, w, M, 3 * kv.d, K, qkv, 3 * kv.d, 1, kv, s);
  return launch_pp<EPI_QKV, 64>(x, w, M, 3 * kv.d, K, qkv, 3 * kv.d, 1, kv, s);
}

}  // namespace ams
