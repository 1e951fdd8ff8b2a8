// Tile plan of the token passes' fp16 GEMMs (more than 64 tokens): plain host
// arithmetic, shared by the launcher, the workspace layout and the CPU tests.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace ams {

// Tile shapes (tokens x weight rows); see gemm_tokens.hip.
enum TokTile {
  TT_256x256 = 0, TT_128x256, TT_256x128, TT_128x128x2, TT_128x128, TT_64x128, TT_128x64, TT_64x256, TT_COUNT
};
struct TokTileInfo {
  int bm, bn, per_cu;  // per_cu: workgroups a CU holds (LDS)
  float one, full;     // us per K step of 64 with one workgroup on the CU, and with all it holds
};
// Measured on the 7B shapes (K = 4096, weights past the caches) with one round of
// workgroups on the CUs; 256 x 256 over many rounds (the clock drops under it).
constexpr TokTileInfo TOK_TILES[TT_COUNT] = {
    {256, 256, 1, 1.50f, 1.60f}, {128, 256, 1, 1.00f, 1.08f}, {256, 128, 1, 1.00f, 1.08f}, {128, 128, 2, 0.75f, 0.98f},
    {128, 128, 1, 0.62f, 0.62f}, {64, 128, 2, 0.52f, 0.82f},  {128, 64, 1, 0.41f, 0.41f},  {64, 256, 1, 0.72f, 0.72f},
};

// K splits of a residual projection (N weight rows, K inputs) of a pass of M > 64
// tokens: its sums run over this many equal ranges of K steps, each from zero, added
// in order.  They are part of the result (h is fp32, its norm rounds to fp16), so they
// follow the shape alone and not the tile that computes it: K is cut until tiles of
// 256 x 256 times splits reach about 256 workgroups, each range at least 8 steps of 64.
inline int tok_resid_splits(int M, int N, int K) {
  if (M <= 64 || N % 256 != 0 || K % 64 != 0) return 1;
  const int tiles = (N / 256) * ((M + 255) / 256);
  if (tiles >= 160) return 1;
  return std::max(1, std::min((256 + tiles - 1) / tiles, (K / 64) / 8));
}

// Tile shape of weight rows 0 .. main_n - 1 (all N of them where rest_tile is
// -1) and of the rest; splits: workgroups along K, each writing its range's sums; or
// segs > 1: one workgroup adds that many ranges itself.
struct TokPlan {
  int tile = TT_128x128, splits = 1, main_n = 0, rest_tile = -1, segs = 1;
  float us = 1e30f;  // modelled
};

// The tile shape of the smallest modelled time: rounds of workgroups over the 256
// CUs times the K steps of one.  The sums are the same on every tile (K order).
//
// S > 1 (a residual projection's ranges): either a workgroup per range writes its
// partial sums for the reduction that adds them (which also applies the next norm), or
// one workgroup runs through all ranges and a norm launch follows (the
// 256 x 256 tile has no registers for the second accumulator).  room: floats there
// are for partial sums.  On 26 O and down shapes of d = 1024, 2048 and 4096 at 72 to
// 2,240 tokens the plan was within 5% of the fastest of both forms on every tile
// (2,240 tokens of d = 1024, K = 4,096 in 8 ranges: 48 us with the norm, 57 us with
// partial sums; 128 tokens of d = 4096, K = 11,008 in 16: 40 us with partial sums, 77 without).
//
// Otherwise, 256 x 256 tiles may keep to the weight rows that fill whole
// rounds and leave the rest to smaller tiles in a second launch (mixed): at 1,024 tokens
// the 7B gate|up projection's 344 tiles are 256 in one round and 88 more tiles'
// work on 352 workgroups of 128 x 128.
inline TokPlan tok_plan(int M, int N, int K, int S, bool mixed, size_t room = SIZE_MAX) {
  TokPlan best;
  const bool parts = S == 1 || (size_t)S * M * N <= room;
  M = (M + 63) / 64 * 64;
  const int kt = K / 64;
  auto rounds_us = [&](const TokTileInfo& i, long wgs, float steps) {
    const long cap = 256L * i.per_cu, full = wgs / cap, rest = wgs - full * cap;
    float t = 3.f + (full + (rest > 0)) * 2.f + full * steps * i.full;
    if (rest > 0) t += steps * (rest <= 256 ? i.one : i.full);
    return t;
  };
  for (int t = 0; t < TT_COUNT; ++t) {
    const TokTileInfo& i = TOK_TILES[t];
    if (N % i.bn != 0) continue;
    const long tm = (M + i.bm - 1) / i.bm, tiles = N / i.bn * tm;
    float us = rounds_us(i, tiles * S, (float)((kt + S - 1) / S)) +
               (S > 1 ? S : 0) * (float)M * N * 4.f / 2.0e6f;  // partial sums written and read back
    if (parts && us < best.us) best = TokPlan{t, S, N, -1, 1, us};
    if (S > 1 && t != TT_256x256) {
      us = rounds_us(i, tiles, (float)kt) + 3.f;
      if (us < best.us) best = TokPlan{t, 1, N, -1, S, us};
    }
    const int main_n = (int)(tiles / 256 * 256 / tm) * i.bn;
    if (!mixed || S > 1 || t != TT_256x256 || main_n == 0 || main_n == N) continue;
    const TokPlan r = tok_plan(M, N - main_n, K, 1, false);
    us = rounds_us(i, main_n / i.bn * tm, (float)kt) + r.us;
    if (us < best.us) best = TokPlan{t, 1, main_n, r.tile, 1, us};
  }
  return best;
}
inline TokPlan tok_resid_plan(int M, int N, int K, size_t room = SIZE_MAX) {
  return tok_plan(M, N, K, tok_resid_splits(M, N, K), false, room);
}

// Floats of partial sums the residual projections (N outputs, K inputs) of passes
// of up to T tokens may need: the splits do not change within a multiple of 256 tokens.
inline size_t tok_part_floats(int N, int K, int T) {
  size_t best = 0;
  for (int M = 256; M < T + 256; M += 256) {
    const int m = std::min(M, T), s = tok_resid_splits(m, N, K);
    if (s > 1) best = std::max(best, (size_t)s * m * N);
    if (m > 64 && (N / 256) * (long)((m + 255) / 256) >= 160) break;
  }
  return best;
}

}  // namespace ams
