// Two-phase hashing for the action index (paper section 3.2.3, "Virtual Action",
// Algorithm 1 "Two-Phase Hashing for Action Index") and the page keys of
// prefixes built on it.
//
// Phase 1 hashes every s-byte segment of the input on its own, phase 2 merges
// the segment hashes in order.  Both hash functions are polynomial hashes
// modulo the Mersenne prime 2^31 - 1, evaluated with two independent bases
// whose 31-bit results are packed into one 64-bit value (first base low):
//   HashFunc1(B_i) = (sum_j u_j r^(s/2-1-j)) r + |B_i|, u_j the 16-bit
//                    little-endian units of B_i zero-padded to s bytes;
//   HashFunc2(h_1..h_k) = (sum_i h_i q^(k-i)) q + N.
//
// Phase 1: a group of G lanes per segment (G = 64, or the power of two that
// holds a shorter segment's 16-byte chunks).  HashFunc1 is a dot product of
// the units with powers of r, and a 16-bit unit times a 31-bit power leaves 17
// bits of headroom in 64: a lane keeps the 8 powers of its place in a round of G
// chunks per base in registers, sums its 8 products without reducing, folds
// rounds with one multiplication by r^(8 G) each, and the group adds the lanes'
// residues.  Bound by HBM and the 64-bit multiply-adds (16 per 16 bytes)
// alike; with a Horner chain per 16 bytes and a tree of modular products per
// segment it was bound by integer ALU: 157 MB in 4 KB segments 209 -> 38 us.
#include <algorithm>
#include <mutex>

#include "common.h"
#include "kernels.h"

namespace ams {

namespace {

constexpr uint64_t M31 = 0x7FFFFFFFull;
constexpr uint32_t HR0 = 0x2545F491u, HR1 = 0x1B873593u;  // HashFunc1 bases
constexpr uint32_t HQ0 = 0x3C6EF372u, HQ1 = 0x0A54FF53u;  // HashFunc2 bases

__device__ __forceinline__ uint64_t red(uint64_t x) {  // x < 2^63 -> x mod (2^31 - 1)
  x = (x & M31) + (x >> 31);
  x = (x & M31) + (x >> 31);
  return x >= M31 ? x - M31 : x;
}
__device__ __forceinline__ uint64_t mulm(uint64_t a, uint64_t b) { return red(a * b); }  // a, b < 2^31
__device__ __forceinline__ uint64_t addm(uint64_t a, uint64_t b) { return red(a + b); }
// b0^e and b1^e, the two chains side by side
__device__ __forceinline__ void powm2(uint64_t b0, uint64_t b1, uint32_t e, uint64_t& r0, uint64_t& r1) {
  r0 = r1 = 1;
  for (; e; e >>= 1) {
    if (e & 1) {
      r0 = mulm(r0, b0);
      r1 = mulm(r1, b1);
    }
    b0 = mulm(b0, b0);
    b1 = mulm(b1, b1);
  }
}

__host__ __device__ constexpr uint64_t pow31(uint64_t b, uint64_t e) {  // b^e mod 2^31 - 1
  uint64_t r = 1;
  for (b %= M31; e; e >>= 1, b = b * b % M31)
    if (e & 1) r = r * b % M31;
  return r;
}

// a + b mod 2^31 - 1 as a value <= 2^31 - 1, for such a and b
__device__ __forceinline__ uint32_t fold_add(uint32_t a, uint32_t b) {
  const uint32_t t = a + b;
  return (t & (uint32_t)M31) + (t >> 31);
}

// Phase 1.  Segment g covers bytes [g s, g s + s) of data (zero beyond
// n_bytes); s is a multiple of 16 and data is 16-byte aligned.  A segment's
// C = s / 16 chunks sit right-aligned in its R rounds of G, so that the lanes
// before its start contribute the polynomial's leading zeros.  m0 / m1 =
// r^(8 G) of the two bases.
__global__ __launch_bounds__(256) void k_hash_segments(const uint8_t* __restrict__ data, uint64_t n_bytes, int s,
                                                       uint64_t k, int G, uint32_t m0, uint32_t m1,
                                                       uint64_t* __restrict__ seg_out) {
  const int lane = threadIdx.x & 63, gl = lane & (G - 1), per = 64 / G;
  const int C = s / 16, R = (C + G - 1) / G, lead = R * G - C;
  uint32_t w0[8], w1[8];  // unit i of the lane's chunk in a segment's last round: r^(8 (G - gl) - i)
  {
    uint64_t a, b;
    powm2(HR0, HR1, 8 * (G - gl) - 7, a, b);
#pragma unroll
    for (int i = 7; i >= 0; --i) {
      w0[i] = (uint32_t)a;
      w1[i] = (uint32_t)b;
      a = mulm(a, HR0);
      b = mulm(b, HR1);
    }
  }
  const uint64_t wave = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6), waves = (uint64_t)gridDim.x * 4;
  for (uint64_t g0 = wave * per; g0 < k; g0 += waves * per) {
    const uint64_t g = g0 + lane / G, base = g * (uint64_t)s;
    uint64_t a0 = 0, a1 = 0;
    for (int rd = 0; rd < R; rd += 4) {
      uint4 q[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int c = (rd + x) * G + gl - lead;
        q[x] = uint4{0u, 0u, 0u, 0u};
        if (rd + x < R && c >= 0 && g < k) {
          const uint64_t off = base + 16ull * c;
          if (off + 16 <= n_bytes) {
            q[x] = *reinterpret_cast<const uint4*>(data + off);
          } else if (off < n_bytes) {  // the input's last bytes
            uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int i = 0; i < 15; ++i)
              if (off + i < n_bytes) w[i >> 2] |= (uint32_t)data[off + i] << (8 * (i & 3));
            q[x] = uint4{w[0], w[1], w[2], w[3]};
          }
        }
      }
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        if (rd + x >= R) break;
        if (rd + x > 0) {  // residues < 2^31 times m < 2^31, plus 8 products < 2^47: below 2^63
          a0 = red(a0) * m0;
          a1 = red(a1) * m1;
        }
        const uint32_t u[4] = {q[x].x, q[x].y, q[x].z, q[x].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t lo = u[i] & 0xFFFFu, hi = u[i] >> 16;
          a0 += (uint64_t)lo * w0[2 * i];
          a0 += (uint64_t)hi * w0[2 * i + 1];
          a1 += (uint64_t)lo * w1[2 * i];
          a1 += (uint64_t)hi * w1[2 * i + 1];
        }
      }
    }
    uint32_t v0 = (uint32_t)red(a0), v1 = (uint32_t)red(a1);
    for (int o = 1; o < G; o <<= 1) {
      v0 = fold_add(v0, __shfl_xor(v0, o, 64));
      v1 = fold_add(v1, __shfl_xor(v1, o, 64));
    }
    if (gl == 0 && g < k) {
      const uint64_t len = n_bytes - base < (uint64_t)s ? n_bytes - base : (uint64_t)s;
      seg_out[g] = red((uint64_t)v0 + len) | (red((uint64_t)v1 + len) << 32);
    }
  }
}

// Phase 2 over k segment hashes, one workgroup of T threads: thread t runs
// Horner over segments t, t + T, ... of a right-aligned index space (neighbouring
// threads read neighbouring hashes; qn0 / qn1 = q^T of the two bases), its sum is
// then worth q^(T - t), and the residues are added.  H = sum + n_bytes per
// component.  (A contiguous range per thread of 256 read 8 bytes per cache line
// and step: 55 -> 17 us for 38,400 segments, most of it one CU's 307 KB of loads.)
constexpr int MERGE_MAX_T = 1024;
__global__ __launch_bounds__(MERGE_MAX_T) void k_hash_merge(const uint64_t* __restrict__ seg, uint64_t k,
                                                            uint64_t n_bytes, uint32_t qn0, uint32_t qn1,
                                                            uint64_t* __restrict__ out) {
  __shared__ uint32_t s0[MERGE_MAX_T / 64], s1[MERGE_MAX_T / 64];
  const int t = threadIdx.x, T = blockDim.x;
  const uint64_t m = (k + T - 1) / T, lead = T * m - k;
  uint64_t a0 = 0, a1 = 0;
  for (uint64_t j = 0; j < m; j += 8) {
    uint64_t h[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const uint64_t vi = (j + x) * T + t;
      h[x] = j + x < m && vi >= lead ? seg[vi - lead] : 0ull;
    }
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      if (j + x >= m) break;
      a0 = red(a0) * qn0 + (h[x] & 0xFFFFFFFFull);
      a1 = red(a1) * qn1 + (h[x] >> 32);
    }
  }
  uint64_t p0, p1;
  powm2(HQ0, HQ1, T - t, p0, p1);
  uint32_t v0 = (uint32_t)mulm(red(a0), p0), v1 = (uint32_t)mulm(red(a1), p1);
  for (int o = 1; o < 64; o <<= 1) {
    v0 = fold_add(v0, __shfl_xor(v0, o, 64));
    v1 = fold_add(v1, __shfl_xor(v1, o, 64));
  }
  if ((t & 63) == 0) {
    s0[t >> 6] = v0;
    s1[t >> 6] = v1;
  }
  __syncthreads();
  if (t == 0) {
    uint64_t h0 = red(n_bytes % M31), h1 = h0;
    for (int w = 0; w < T / 64; ++w) {
      h0 = addm(h0, s0[w]);
      h1 = addm(h1, s1[w]);
    }
    out[0] = h0 | (h1 << 32);
  }
}

// Page keys of packed rows: row b spans row_bytes[b] bytes whose segment
// hashes (the row's bytes start on a segment boundary) sit from seg +
// seg_first[b] on.  Key of page m (m < floor(row_bytes / page_bytes)) =
// HashFunc2 of the row's segments covering its first (m + 1) page_bytes bytes.
// One thread per row (a sequential scan of a few hundred segments).
__global__ void k_hash_page_keys(const uint64_t* __restrict__ seg, const int64_t* __restrict__ seg_first,
                                 const int64_t* __restrict__ row_bytes, int B, int64_t page_bytes, int s,
                                 int max_pages, uint64_t* __restrict__ keys) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const int64_t per_page = page_bytes / s, n_pages = min<int64_t>(row_bytes[b] / page_bytes, max_pages);
  const uint64_t* sg = seg + seg_first[b];
  uint64_t a0 = 0, a1 = 0;
  for (int64_t pg = 0; pg < n_pages; ++pg) {
    for (int64_t i = pg * per_page; i < (pg + 1) * per_page; ++i) {
      a0 = addm(mulm(a0, HQ0), sg[i] & 0xFFFFFFFFull);
      a1 = addm(mulm(a1, HQ1), sg[i] >> 32);
    }
    const uint64_t len = red((uint64_t)((pg + 1) * page_bytes) % M31);
    keys[(size_t)b * max_pages + pg] = addm(mulm(a0, HQ0), len) | (addm(mulm(a1, HQ1), len) << 32);
  }
}

}  // namespace

// Scratch of the allocation-free index hash (ams_index_hash_noalloc): the
// phase-1 segment hashes of one call, at most INDEX_NOALLOC_MAX_SEGMENTS of
// them (1 MiB).  Every device the library runs on holds its own copy until the
// process ends, and every call on that device shares it.  Host code never
// passes the array's name to a kernel: it takes the device address that
// hipGetSymbolAddress returned for the current device (index_noalloc_scratch).
static __device__ __align__(256) uint64_t scratch[INDEX_NOALLOC_MAX_SEGMENTS];

namespace {
std::mutex g_scratch_mu;
uint64_t* g_scratch_ptr[64] = {};  // per device id
}  // namespace

hipError_t index_noalloc_scratch(int device, uint64_t** ptr) {
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (device < 0 || device >= 64) return hipErrorInvalidDevice;
  if (!g_scratch_ptr[device]) {  // once per device, with that device current
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = (uint64_t*)p;
  }
  *ptr = g_scratch_ptr[device];
  return hipSuccess;
}

hipError_t hash_segments(const void* data, uint64_t n_bytes, int s, uint64_t* seg_out, hipStream_t st) {
  const uint64_t k = (n_bytes + s - 1) / s;
  if (k == 0) return hipSuccess;
  int G = 64;
  while (G > 1 && G / 2 >= s / 16) G /= 2;
  const uint64_t per_wg = 4 * (64 / G);  // segments of a workgroup's pass
  const uint64_t wgs = std::min<uint64_t>((k + per_wg - 1) / per_wg, 2048);  // 8 per CU resident
  hipLaunchKernelGGL(k_hash_segments, dim3((unsigned)wgs), dim3(256), 0, st, (const uint8_t*)data, n_bytes, s, k, G,
                     (uint32_t)pow31(HR0, 8 * G), (uint32_t)pow31(HR1, 8 * G), seg_out);
  return hipGetLastError();
}

hipError_t hash_merge(const uint64_t* seg, uint64_t k, uint64_t n_bytes, uint64_t* out, hipStream_t st) {
  int T = 64;  // few segments: few waves to start and join
  while (T < MERGE_MAX_T && (uint64_t)T < k) T *= 2;
  hipLaunchKernelGGL(k_hash_merge, dim3(1), dim3(T), 0, st, seg, k, n_bytes, (uint32_t)pow31(HQ0, T),
                     (uint32_t)pow31(HQ1, T), out);
  return hipGetLastError();
}

hipError_t hash_page_keys(const uint64_t* seg, const int64_t* seg_first, const int64_t* row_bytes, int B,
                          int64_t page_bytes, int s, int max_pages, uint64_t* keys, hipStream_t st) {
  hipLaunchKernelGGL(k_hash_page_keys, dim3((B + 63) / 64), dim3(64), 0, st, seg, seg_first, row_bytes, B,
                     page_bytes, s, max_pages, keys);
  return hipGetLastError();
}

}  // namespace ams
