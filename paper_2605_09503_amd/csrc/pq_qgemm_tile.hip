// Which output tile the product kernels take for a shape (host code).
#include "pq_qgemm_common.h"

namespace pq {

// The tile with the shortest predicted time of `problems` products of that shape in one launch.  n workgroups run on 256
// compute units, each does s 64-wide steps; with c = ceil(n / 256) rounds and r = max(n / 256, 1) of them really filled,
//     time = l0 + odd (N mod 8) + max(rounds (a + b s), l1 s),  rounds = th c + (1 - th) r,
// where l1 s is the latency of one workgroup's chain of steps in the tiles whose workgroups share a unit, and odd the
// stores of the columns past the last whole eight, one by one in the workgroups of the right edge (3.5 to 10 us of a
// 256-row tile at N mod 8 = 7: without that term INT3 g64 2892 x 2765 x 832 took the 224-row tile at 26.6 us; 64 x 64
// takes 21.7).
// The coefficients (us) are least-squares fits of the logarithm of measured times, graph replays, over 1285 shapes of
// 1e7 to 7e11 operations: NVFP4 303, INT4 and INT3 982 with groups of 32, 64, 128 and 256, 16 to 8192 rows, 128 to 12288
// columns, K 96 to 12288, a quarter of them round sizes, half of them where a round of large tiles is partly or
// just filled; then moved by at most 4 % a tile so that the choices cost least.  They were fitted with four waves a 64 x 64
// and 64 x 96 tile, to single products: what eight waves take (below) and launches of several problems is not in them.
// Measured with the kernels as they are, all tiles of 10900 random shapes of these ranges, packed: the choice costs 0.54 %
// over the best tile in the mean, more than 5 % for 4.3 % of them, at most 21 % (INT4 g32 132 x 11376 x 160, 128 x 128 8.9 us, 64 x
// 64 7.3).  Where the line lies, e.g. NVFP4, K = 3072 (split 64 x 96 | 256 or 224 x 256, us):
// 1024 x 3072 22 | 30 (of 128 x 128), 2048 x 3072 41 | 47, 4608 x 3072 92 | 79.
struct TileCost {
  float a, b, l0, l1, th, odd;
};
struct TileSize {
  int bm, bn;
};
static constexpr TileSize kTileSize[] = {{0, 0}, {256, 256}, {128, 128}, {224, 256}, {32, 32}, {64, 32}, {64, 64}, {64, 96}, {64, 64}, {64, 96}};
// rows: NVFP4; INT4 and INT3 with groups of 32; INT4 with larger groups; INT3 with larger groups.  Columns: the tiles in
// the order of their numbers.
static constexpr TileCost kTileCost[4][8] = {
    {{}, {9.46f, 1.347f, 0.0f, 0.0f, 1.0f, 1.4f}, {1.98f, 0.498f, 4.94f, 0.637f, 0.632f, 0.44f}, {9.17f, 1.283f, 0.0f, 0.0f, 0.858f, 1.2f},
     {0.511f, 0.05455f, 3.35f, 0.0635f, 0.899f, 0.0f}, {1.06f, 0.07814f, 2.85f, 0.0949f, 0.929f, 0.0f}, {1.1f, 0.1194f, 3.85f, 0.168f, 0.762f, 0.079f},
     {2.13f, 0.166f, 4.01f, 0.219f, 0.681f, 0.091f}},
    {{}, {9.68f, 1.416f, 0.0f, 0.0f, 0.964f, 1.3f}, {2.13f, 0.537f, 4.19f, 0.66f, 0.593f, 0.54f}, {9.92f, 1.362f, 0.0f, 0.0f, 0.794f, 0.96f},
     {0.501f, 0.06657f, 3.24f, 0.0619f, 0.841f, 0.0f}, {1.03f, 0.09627f, 2.85f, 0.116f, 0.868f, 0.0f}, {1.11f, 0.1401f, 3.89f, 0.184f, 0.71f, 0.05f},
     {1.92f, 0.1927f, 4.15f, 0.229f, 0.808f, 0.12f}},
    {{}, {10.0f, 1.305f, 1.33f, 0.0f, 0.975f, 1.1f}, {2.17f, 0.5552f, 4.14f, 0.696f, 0.645f, 0.49f}, {9.03f, 1.195f, 1.93f, 0.0f, 0.949f, 0.93f},
     {0.5f, 0.06711f, 3.21f, 0.0f, 0.915f, 0.0f}, {1.04f, 0.09957f, 2.85f, 0.0f, 0.813f, 0.0f}, {1.09f, 0.1439f, 3.9f, 0.176f, 0.832f, 0.065f},
     {1.97f, 0.1987f, 4.39f, 0.235f, 0.662f, 0.11f}},
    {{}, {9.96f, 0.9593f, 0.0f, 0.0f, 0.947f, 1.4f}, {2.18f, 0.5174f, 3.71f, 0.858f, 0.616f, 0.55f}, {9.34f, 0.8692f, 0.0f, 0.0f, 0.893f, 1.2f},
     {0.609f, 0.03245f, 3.26f, 0.0435f, 0.744f, 0.0f}, {1.1f, 0.04921f, 2.92f, 0.0676f, 0.699f, 0.0f}, {1.28f, 0.07574f, 3.61f, 0.201f, 0.75f, 0.065f},
     {2.32f, 0.1103f, 4.02f, 0.176f, 0.698f, 0.038f}},
};

// Whether eight waves and not four share a tile of 64 x 64 or 64 x 96: where no unit has a second workgroup to run beside
// the first, and each wave has a few steps.  A wave issues a vector instruction every five cycles at most, so one wave a SIMD
// leaves half of the vector unit idle and two do not.  Both layouts take the sums in one order, so a
// line is one for both; where a few steps more let packed operands gain and row-major ones not yet, it lies between.
// Shapes of 112 to 256 tiles, eight against four, medians by steps of K (NVFP4, integer, INT3 codes):
//   packed       24: 1.03 1.03 1.02   28: 1.00 1.01 0.98   36: 0.98 1.00 0.95   48: 0.96 0.99 0.93   70: 0.94 0.96 0.88
//   row-major, rows that start at a line of the cache (K a multiple of 256), through LDS (split_eight)
//                24: 0.80 1.00 1.00   28: 0.94 1.02 1.03   36: 0.91 1.02 1.02   48: 0.75 0.92 0.90   70: 0.75 0.83 0.77
//   other rows   24: 1.01 1.03        28: 1.02 1.05 1.02   36: 0.94 1.05 1.06   48: 0.88 1.03 0.87   70: 0.81 0.98, up to 1.07
// (sets of eight steps: multiples of eight are the good ones).  With the lines as here 2700 packed shapes take 0.955 of the
// time of four waves throughout (16 above 1.02), 2600 row-major ones 0.89 (70 above 1.02, at most 1.10: INT4 g128 1712 x 356
// x 4224 17.7 -> 19.4 us).  With 512 and 768 tiles 1.15: the second workgroup covers the first one's ends.  Sixteen waves for the
// smaller tiles: 0.96 to 1.23.
static bool split_eight_waves(int cls, int64_t n_tiles, int64_t K) {
  const bool lines = K % 256 == 0;
  const int steps = cls == 0 ? (lines ? 24 : 36) : cls == 3 ? (lines ? 28 : 44) : lines ? 36 : 56;
  return n_tiles <= 256 && K > steps * kBK;
}

// A call of several launches takes one choice for all of them: the tile and its waves fix the order of the sums over K.
int choose_tile(pq_format fmt, int group, int64_t M, int64_t N, int64_t K, int problems) {
  const int cls = fmt == PQ_FMT_NVFP4 ? 0 : group == 32 ? 1 : fmt == PQ_FMT_INT4 ? 2 : 3;
  const float s = (float)((K + kBK - 1) / kBK), past = (float)(N % 8);
  int best = kTile256;
  float best_t = 0.0f;
  for (int t = kTile256; t <= kTileSplit64x96; ++t) {
    const TileCost& k = kTileCost[cls][t];
    const TileSize& z = kTileSize[t];
    const int64_t n = ((M + z.bm - 1) / z.bm) * ((N + z.bn - 1) / z.bn) * problems;
    const float c = (float)((n + 255) / 256), r = n > 256 ? (float)n / 256.0f : 1.0f;
    float time = (k.th * c + (1.0f - k.th) * r) * (k.a + k.b * s);
    if (time < k.l1 * s) time = k.l1 * s;
    time += k.l0 + k.odd * past;
    if (t == kTile256 || time < best_t) {
      best = t;
      best_t = time;
    }
  }
  if (best == kTileSplit64 || best == kTileSplit64x96) {
    if (split_eight_waves(cls, qgemm_tiles(best, M, N) * problems, K)) best = best == kTileSplit64 ? kTileSplit64Eight : kTileSplit64x96Eight;
  }
  return best;
}

void tile_size(int tile, int* bm, int* bn) {
  *bm = kTileSize[tile].bm;
  *bn = kTileSize[tile].bn;
}

int tile_waves(int tile) { return tile == kTile128 || tile == kTileSplit64 || tile == kTileSplit64x96 ? 4 : 8; }

int64_t qgemm_tiles(int tile, int64_t M, int64_t N) {
  const TileSize& z = kTileSize[tile];
  return ((M + z.bm - 1) / z.bm) * ((N + z.bn - 1) / z.bn);
}

}  // namespace pq
