// Tile plan of the token passes' fp16 GEMMs (more than 64 tokens): plain host
// arithmetic, shared by the launcher, the workspace layout and the CPU tests.
#pragma once

#include <algorithm>
#include <cstddef>

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
    {256, 256, 1, 1.50f, 1.60f}, {128, 256, 1, 1.00f, 1.08f}, {256, 128, 1, 1.00f, 1.08f}, {128, 128, 2, 0.85f, 1.06f},
    {128, 128, 1, 0.62f, 0.62f}, {64, 128, 2, 0.52f, 0.82f},  {128, 64, 1, 0.44f, 0.44f},  {64, 256, 1, 0.72f, 0.72f},
};

// Tile shape of weight rows 0 .. main_n - 1 (all N of them where rest_tile is
// -1) and of the rest, and the K splits.
struct TokPlan {
  int tile = TT_128x128, splits = 1, main_n = 0, rest_tile = -1;
  float us = 1e30f;  // modelled
};

// The tile shape (and, with split, the K splits) of the smallest modelled time:
// rounds of workgroups over the 256 CUs times the K steps of one, plus what a
// split's partial sums cost in the reduction that adds them.  On the shapes of
// d = 1024, 2048 and 4096 decoders at 72 to 19,200 tokens the plan was the
// fastest of the measured tiles and splits or within 8% of it.
//
// Without splits, 256 x 256 tiles may keep to the weight rows that fill whole
// rounds and leave the rest to smaller tiles in a second launch: at 1,024 tokens
// the 7B gate|up projection's 344 tiles are 256 in one round and 88 more tiles'
// work on 352 workgroups of 128 x 128.
inline TokPlan tok_plan(int M, int N, int K, bool split, bool mixed = true) {
  TokPlan best;
  M = (M + 63) / 64 * 64;  // one plan per 64 tokens (tok_part_floats)
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
    const int smax = split ? std::max(1, std::min(16, kt / 8)) : 1;
    for (int s = 1; s <= smax; ++s) {
      if (s > 1 && tiles * s > 1024) break;
      const float us = rounds_us(i, tiles * s, (float)((kt + s - 1) / s)) +
                       (s > 1 ? s : 0) * (float)M * N * 4.f / 3.0e6f;  // partial sums written and read back
      if (us < best.us) best = TokPlan{t, s, N, -1, us};
    }
    const int main_n = (int)(tiles / 256 * 256 / tm) * i.bn;
    if (split || !mixed || t != TT_256x256 || main_n == 0 || main_n == N) continue;
    const TokPlan r = tok_plan(M, N - main_n, K, false, false);
    const float us = rounds_us(i, main_n / i.bn * tm, (float)kt) + r.us;
    if (us < best.us) best = TokPlan{t, 1, main_n, r.tile, us};
  }
  return best;
}

// Floats of split-K partial sums the residual projections (N outputs, K inputs)
// of token passes of up to T tokens need: the plan's splits do not change
// within a multiple of 64 tokens.
inline size_t tok_part_floats(int N, int K, int T) {
  size_t best = 0;
  for (int M = 128; M < T + 64; M += 64) {
    const int m = std::min(M, T);
    if (m <= 64 || (N % 256 == 0 && (long)(N / 256) * (m / 256) > 512)) break;  // (past that no plan splits)
    const int s = tok_plan(m, N, K, true).splits;
    if (s > 1) best = std::max(best, (size_t)s * m * N);
  }
  return best;
}

}  // namespace ams
