// Test-only C ABI over single kernels (libams_probe.so), used by the GPU
// kernel tests to check one launcher at a time against plain definitions.
// Not part of the product library; the decoder's ABI is include/ams.h.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"

namespace {

// One thread per 16 bytes of W [N][K] (K a multiple of 32) in fragment order.
__global__ void k_pack(const uint4* W, int N, int K, uint4* Wf) {
  const size_t o = (size_t)blockIdx.x * blockDim.x + threadIdx.x, ks = K / 32;
  if (o >= (size_t)N * K / 8) return;
  const size_t l = o & 63, blk = o >> 6;
  Wf[o] = W[((blk / ks) * 16 + (l & 15)) * (K / 8) + (blk % ks) * 4 + (l >> 4)];
}

// The row-major weights of a probe call in the order the token GEMMs read.
struct Packed {
  void* p = nullptr;
  hipStream_t s;
  Packed(const void* W, int N, int K, hipStream_t st) : s(st) {
    if (N % 16 || K % 32 || hipMalloc(&p, (size_t)N * K * 2) != hipSuccess) return;
    hipLaunchKernelGGL(k_pack, dim3((unsigned)(((size_t)N * K / 8 + 255) / 256)), dim3(256), 0, s, (const uint4*)W, N, K,
                       (uint4*)p);
  }
  ~Packed() {
    (void)hipStreamSynchronize(s);
    (void)hipFree(p);
  }
  template <typename F> int run(F f) {
    if (!p) return (int)hipErrorInvalidValue;
    const hipError_t e = hipGetLastError();
    return (int)(e == hipSuccess ? f() : e);
  }
};

}  // namespace

extern "C" {

int ams_probe_gemm(int dtype, int epi, const void* u, const void* ulo, const void* W, int M, int N, int K, void* out,
                   int ldo, void* o16, void* olo, void* stream) {
  if (dtype == ams::DT_F16 && M > 64 && !ulo && !o16 && !olo) {  // a token pass
    Packed w(W, N, K, (hipStream_t)stream);
    return w.run([&] { return ams::gemm_tokens(epi, u, w.p, M, N, K, out, ldo, w.s); });
  }
  return (int)ams::gemm(dtype, epi, u, W, M, N, K, out, ldo, (hipStream_t)stream, ulo, o16, olo);
}

int ams_probe_gemv_f32(int epi, const float* x, int norm, float eps, const float* W, int M, int N, int K, float* out,
                       int ldo, int splits, float* part, unsigned* cnt, void* stream) {
  return (int)ams::gemv_f32(epi, x, norm != 0, eps, W, M, N, K, out, ldo, (hipStream_t)stream, splits, part, cnt);
}

// a token GEMM on one tile shape, weights in fragment order
int ams_probe_gemm_tokens(int tile, int epi, const void* u, const void* Wf, int M, int N, int K, void* out, int ldo,
                          int splits, void* stream) {
  return (int)ams::gemm_tokens_tile(tile, epi, u, Wf, M, N, K, out, ldo, splits, (hipStream_t)stream);
}
// a residual projection whose K ranges one workgroup per tile adds
int ams_probe_gemm_tokens_segs(int tile, const void* u, const void* Wf, int M, int N, int K, float* h, int segs,
                               void* stream) {
  return (int)ams::gemm_tokens_tile(tile, ams::EPI_RESID, u, Wf, M, N, K, h, N, 1, (hipStream_t)stream, segs);
}
int ams_probe_gemm_tokens_short(int epi, const void* u, const void* Wf, int M, int N, int K, void* out, int ldo,
                                void* stream) {
  return (int)ams::gemm_tokens_short(epi, u, Wf, M, N, K, out, ldo, (hipStream_t)stream);
}
int ams_probe_tok_resid_splits(int M, int N, int K) { return ams::tok_resid_splits(M, N, K); }
// out[0..3]: tile, splits, weight rows on it, tile of the rest (-1: none)
void ams_probe_tok_plan(int M, int N, int K, int split, int32_t* out) {
  const ams::TokPlan p = split ? ams::tok_resid_plan(M, N, K) : ams::tok_plan(M, N, K, 1, true);
  out[0] = p.tile; out[1] = p.splits; out[2] = p.main_n; out[3] = p.rest_tile;
}
size_t ams_probe_tok_part_floats(int N, int K, int T) { return ams::tok_part_floats(N, K, T); }

int ams_probe_gemm_big(int epi, const void* u, const void* W, int M, int N, int K, void* out, int ldo, int bn,
                       void* stream) {
  const int tile = bn == 256 ? ams::TT_256x256 : bn == 128 ? ams::TT_256x128 : ams::TT_128x64;
  Packed w(W, N, K, (hipStream_t)stream);
  return w.run([&] { return ams::gemm_tokens_tile(tile, epi, u, w.p, M, N, K, out, ldo, 1, w.s); });
}

int ams_probe_gemm_big_part(const void* u, const void* W, int M, int N, int K, int splits, float* part,
                            void* stream) {
  Packed w(W, N, K, (hipStream_t)stream);
  return w.run([&] {
    return ams::gemm_tokens_tile(ams::TT_256x256, ams::EPI_PART, u, w.p, M, N, K, part, N, splits, w.s);
  });
}

int ams_probe_gemm_part(const void* u, const void* ulo, const void* W, int M, int N, int K, int splits, float* part,
                        void* stream) {
  return (int)ams::gemm_part(u, ulo, W, M, N, K, splits, part, (hipStream_t)stream);
}

int ams_probe_part_resid(const float* part, int splits, int M, int N, float* h, void* o16, void* olo, void* stream) {
  return (int)ams::part_resid(part, splits, M, N, h, o16, olo, (hipStream_t)stream);
}

int ams_probe_frag_pack(const void* W, int N, int K, void* Wf, void* stream) {
  return (int)ams::frag_pack(W, N, K, Wf, (hipStream_t)stream);
}
int ams_probe_gemm_wide(const void* u, const void* ulo, const void* W, int M, int N, int K, int splits, float* part,
                        void* stream) {
  return (int)ams::gemm_wide(u, ulo, W, M, N, K, splits, part, (hipStream_t)stream);
}

int ams_probe_gemm_wide_reduce(int epi, const void* u, const void* ulo, const void* W, int M, int N, int K,
                               int splits, float* part, unsigned* counters, void* out, void* olo, int ldo, float* h,
                               void* o16, void* olo2, float* ss_out, const float* ss_in, float eps, void* stream) {
  return (int)ams::gemm_wide_reduce(epi, u, ulo, W, M, N, K, splits, part, counters, out, olo, ldo, h, o16, olo2,
                                    ss_out, ss_in, eps, (hipStream_t)stream);
}

int ams_probe_part_store(const float* part, int splits, int M, int N, float* out, void* stream) {
  return (int)ams::part_store(part, splits, M, N, out, (hipStream_t)stream);
}
int ams_probe_part_resid_ss(const float* part, int splits, int M, int N, float* h, void* o16, void* olo, float* ss,
                            void* stream) {
  return (int)ams::part_resid(part, splits, M, N, h, o16, olo, (hipStream_t)stream, ss);
}
int ams_probe_part_store_norm(const float* part, int splits, int M, int N, float* out, const float* ss, int d,
                              float eps, void* stream) {
  return (int)ams::part_store(part, splits, M, N, out, (hipStream_t)stream, ss, d, eps);
}
int ams_probe_part_swiglu_norm(const float* part, int splits, int M, int N, void* out, void* olo, const float* ss,
                               int d, float eps, void* stream) {
  return (int)ams::part_swiglu(part, splits, M, N, out, olo, (hipStream_t)stream, ss, d, eps);
}

int ams_probe_part_swiglu(const float* part, int splits, int M, int N, void* out, void* olo, void* stream) {
  return (int)ams::part_swiglu(part, splits, M, N, out, olo, (hipStream_t)stream);
}

int ams_probe_resid_norm(const float* part, int splits, int M, int d, float* h, float eps, void* u, void* stream) {
  return (int)ams::resid_norm(part, splits, M, d, h, eps, u, (hipStream_t)stream);
}

int ams_probe_rmsnorm(int dtype, const float* h, int M, int d, float eps, void* u, void* ulo, void* stream) {
  return (int)ams::rmsnorm(dtype, h, M, d, eps, u, (hipStream_t)stream, ulo);
}

// feeding with the sums of squares of the fed rows per 128 columns
int ams_probe_argmax_feed_ss(const float* logits, int ld, const void* bin_embed, int B, int d, int n_bins,
                             int32_t* out_tok, float* h, void* h16, void* h16lo, float* ss, void* stream) {
  return (int)ams::argmax_feed(ams::DT_F16, logits, ld, bin_embed, B, d, n_bins, 1, 0, out_tok, nullptr, nullptr, h, 1,
                               (hipStream_t)stream, h16, h16lo, ss);
}
int ams_probe_argmax_feed(int ct, const float* logits, int ld, const void* bin_embed, int B, int d, int n_bins,
                          int A, int j, int32_t* out_tok, float* out_logits, const int32_t* forced, float* h, int feed,
                          void* h16, void* h16lo, void* stream) {
  return (int)ams::argmax_feed(ct, logits, ld, bin_embed, B, d, n_bins, A, j, out_tok, out_logits, forced, h, feed,
                               (hipStream_t)stream, h16, h16lo);
}

int ams_probe_gemv_rmsnorm(int ct, int epi, const void* hhi, const void* hlo, float eps, const void* W, int M, int N,
                           int K, void* out, int ldo, void* o16, void* olo, void* stream) {
  return (int)ams::gemv_rmsnorm(ct, epi, hhi, eps, W, M, N, K, out, ldo, (hipStream_t)stream, hlo, o16, olo);
}

// decode attention of one pass (jpos) for B rows, merged when splits > 1; K/V in
// page pools [page][H][64][dh] with row b's page table at pt + b * (cap / 64)
// (order: NULL or the rows' dispatch order, see len_order)
int ams_probe_attn_decode(int ct, const float* qkv, const int32_t* lens, int jpos, int B, int H, int dh, int cap,
                          const int32_t* pt, int splits, const void* rope, void* kslab, void* vslab, float* part,
                          void* o, void* olo, const int32_t* order, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  hipError_t e = ams::attn_decode(ct, qkv, lens, jpos, B, H, dh, cap, ams::KvPages{pt, cap / 64}, splits,
                                  (const float2*)rope, kslab, vslab, part, o, s, olo, ams::QkvParts{}, order);
  if (e == hipSuccess && splits > 1) e = ams::attn_merge(ct, part, B, H, dh, splits, o, s, olo);
  return (int)e;
}

int ams_probe_len_order(const int32_t* lens, int B, int32_t* order, void* stream) {
  return (int)ams::len_order(lens, B, order, (hipStream_t)stream);
}

// Causal attention of packed segments (row[s], pos[s], off[s..s+1]) over their rows' K/V pages.
int ams_probe_attn_decode_parts(int ct, const float* qpart, int qsplits, const float* ss, int nss, float eps,
                                const int32_t* lens, int jpos, int B, int H, int dh, int cap, const int32_t* pt,
                                int splits, const void* rope, void* kslab, void* vslab, float* part, void* o, void* olo,
                                void* stream) {
  hipStream_t s = (hipStream_t)stream;
  ams::QkvParts qp;
  qp.part = qpart;
  qp.splits = qsplits;
  qp.ss = ss;
  qp.nss = nss;
  qp.eps = eps;
  hipError_t e = ams::attn_decode(ct, qpart, lens, jpos, B, H, dh, cap, ams::KvPages{pt, cap / 64}, splits,
                                  (const float2*)rope, kslab, vslab, part, o, s, olo, qp);
  if (e == hipSuccess && splits > 1) e = ams::attn_merge(ct, part, B, H, dh, splits, o, s, olo);
  return (int)e;
}

// K/V append of a pass's tokens, and the QKV GEMM with the append in its epilogue
// (token tables into tok_base / tok_pos first)
int ams_probe_kv_append(int ct, const float* qkv, const int32_t* row, const int32_t* pos, const int32_t* off,
                        int n_seg, int n_tok, int max_len, int max_end, int H, int dh, int cap, const int32_t* pt,
                        const void* rope, void* kslab, void* vslab, void* stream) {
  ams::Segs sg{row, pos, off, n_seg, n_tok, max_len, max_end};
  return (int)ams::kv_append(ct, qkv, sg, H, dh, ams::KvPages{pt, cap / 64}, (const float2*)rope, kslab, vslab,
                             (hipStream_t)stream);
}
int ams_probe_kv_append_tab(const float* qkv, const int32_t* row, const int32_t* pos, const int32_t* off, int n_seg,
                            int n_tok, int H, int dh, int cap, const int32_t* pt, const void* rope, void* kslab,
                            void* vslab, int64_t* tok_base, int32_t* tok_pos, void* stream) {
  ams::Segs sg{row, pos, off, n_seg, n_tok, 0, 0};
  hipStream_t s = (hipStream_t)stream;
  hipError_t e = ams::tok_tables(sg, ams::KvPages{pt, cap / 64}, H, dh, tok_base, tok_pos, s);
  if (e == hipSuccess) e = ams::kv_append_tab(qkv, n_tok, tok_base, tok_pos, H, dh, (const float2*)rope, kslab, vslab, s);
  return (int)e;
}
int ams_probe_qkv_kv(const void* u, const void* W, int K, float* qkv, const int32_t* row, const int32_t* pos,
                     const int32_t* off, int n_seg, int n_tok, int H, int dh, int cap, const int32_t* pt,
                     const void* rope, void* kslab, void* vslab, int64_t* tok_base, int32_t* tok_pos, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  ams::Segs sg{row, pos, off, n_seg, n_tok, 0, 0};
  ams::KvPages kp{pt, cap / 64};
  hipError_t e = ams::tok_tables(sg, kp, H, dh, tok_base, tok_pos, s);
  if (e != hipSuccess) return (int)e;
  ams::KvEpi kv{tok_base, tok_pos, kslab, vslab, (const float2*)rope, H * dh, dh};
  Packed w(W, 3 * H * dh, K, s);
  return w.run([&] { return ams::gemm_qkv_kv(u, w.p, n_tok, K, qkv, kv, s); });
}
int ams_probe_qkv_fusable(int M, int N, int dh, int d) { return ams::gemm_qkv_fusable(M, N, dh, d) ? 1 : 0; }

int ams_probe_attn_prefill(int ct, const float* qkv, const int32_t* row, const int32_t* pos, const int32_t* off,
                           int n_seg, int n_tok, int max_len, int max_end, int H, int dh, int cap, const int32_t* pt,
                           const void* rope, const void* kslab, const void* vslab, void* o, void* stream) {
  ams::Segs sg{row, pos, off, n_seg, n_tok, max_len, max_end};
  return (int)ams::attn_prefill(ct, qkv, sg, H, dh, ams::KvPages{pt, cap / 64}, (const float2*)rope, kslab, vslab, o,
                                (hipStream_t)stream);
}

// one flow embedding of the latents x into h, then the readout of h into x
int ams_probe_flow(int st, float* x, const void* w_in, const void* w_t, const void* w_out, float tau, float eps, float dt,
                   int n_tok, int a, int d, float* h, void* stream) {
  hipError_t e = ams::flow_embed(st, x, w_in, w_t, tau, n_tok, a, d, h, (hipStream_t)stream);
  if (e == hipSuccess) e = ams::flow_update(st, h, w_out, eps, dt, n_tok, a, d, x, (hipStream_t)stream);
  return (int)e;
}

int ams_probe_stream_copy(const void* src, void* dst, size_t bytes, int grid, void* stream) {
  return (int)ams::stream_copy(src, dst, bytes, grid, (hipStream_t)stream);
}

int ams_probe_stream_read(const void* src, size_t bytes, float* out, int grid, void* stream) {
  return (int)ams::stream_read(src, bytes, out, grid, (hipStream_t)stream);
}

int ams_probe_mfma_loop(int shape, float x, int iters, float* out, int grid, void* stream) {
  return (int)ams::mfma_loop(shape, x, iters, out, grid, (hipStream_t)stream);
}

double ams_probe_mfma_loop_flops(int iters, int grid) { return ams::mfma_loop_flops(iters, grid); }

}  // extern "C"
