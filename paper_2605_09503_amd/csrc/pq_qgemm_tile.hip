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
// The coefficients (us) began as least-squares fits of the logarithm of measured times (graph replays, 1285 shapes of 1e7 to 7e11
// operations, 16 to 8192 rows, 128 to 12288 columns, K 96 to 12288).  Those of the first three rows were then moved, a few
// at a time, wherever that made the choices cost less over random shapes of which the tiles were timed: what they predict are ratios
// of neighbouring tiles, no longer times (the third row by 3100 packed shapes; the first two by 3400 shapes of up to 8e10 operations and some
// 900 of up to 3e12 each, in both layouts, with a price on what was slower than the choices before).  The search kept the tiles that the tests
// ask for.  Over shapes that it had not seen, up to 8e10 operations, the choice costs over the best tile, in the mean (more than 5 %
// for, at most): NVFP4 packed 0.7 % (4.2 %, 28 %), row-major 1.4 % (8 %); groups of 32 0.4 % (2.8 %, 24 %), 0.9 % (6 %); INT4 0.7 % (5 %, 34 %),
// 0.6 % (5 %); INT3 with larger groups, which keeps its first fit, 1.7 % (12 %, 39 %); with the first fits 1.4, 1.7; 1.2, 1.2; 1.4, 0.9 %.
// Where the choice differs from the first fit's (7 to 9 % of the shapes) packed operands take 0.92 to 0.93 of the time, row-major ones 0.96 to 0.97; of 1100
// shapes each 6, 7 and 2 packed ones lose more than 2 %, at most 13 %, and 14 to 16 row-major ones, at most 17 % (NVFP4 37 x 9559 x 1920, the
// kernels as they are: packed 8.7 -> 8.1, row-major 9.2 -> 9.6).  INT4 of 5e10 to 6e11 operations: one tile for both layouts helps the one and costs
// the other, 0.94 and 1.07 on the 8 % of them where it changed.  In single products; a whole selection by output error, whose launches
// hold several, takes 0.95 of the time that it took with the first fits and the kernels of then (60000 shapes, at most 1.08).  Where the line lies, e.g.
// NVFP4, K = 3072 (split 64 x 96 | 256 or 224 x 256, us): 1024 x 3072 22 | 32 (of 128 x 128), 2048 x 3072 37 | 47 (the same), 4608 x 3072 81 | 70.
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
    {{}, {10.27f, 1.11f, 0.4591f, 0.03709f, 1.0f, 2.277f}, {2.149f, 0.4713f, 4.489f, 0.04796f, 0.6695f, 0.5793f}, {9.647f, 1.055f, 0.1511f, 0.06031f, 1.0f, 1.34f},
     {0.6366f, 0.06033f, 3.127f, 0.04826f, 0.3135f, 0.002926f}, {1.126f, 0.07982f, 2.681f, 0.009439f, 0.7159f, 0.01874f}, {1.067f, 0.1055f, 3.549f, 0.1499f, 0.6649f, 0.1685f},
     {1.814f, 0.1478f, 3.781f, 0.02284f, 0.5977f, 0.1431f}},
    {{}, {9.662f, 1.371f, 0.2073f, 0.01711f, 0.9232f, 1.267f}, {2.067f, 0.5588f, 4.283f, 1.133f, 0.8489f, 0.5542f}, {9.772f, 1.246f, 0.1311f, 0.04011f, 1.0f, 1.309f},
     {0.4727f, 0.07413f, 3.301f, 0.06303f, 0.8232f, 0.01681f}, {1.058f, 0.09064f, 2.855f, 0.111f, 0.8681f, 0.001728f}, {1.104f, 0.1389f, 3.774f, 0.1662f, 0.7911f, 0.03378f},
     {1.793f, 0.1908f, 3.921f, 0.2483f, 0.7217f, 0.1146f}},
    {{}, {10.78f, 1.33f, 1.034f, 0.001557f, 1.0f, 1.105f}, {2.17f, 0.5597f, 3.94f, 1.029f, 0.8401f, 0.4839f}, {9.283f, 1.259f, 1.786f, 0.003477f, 1.0f, 0.9902f},
     {0.5175f, 0.07548f, 3.21f, 0.02426f, 0.8443f, 0.0f}, {1.042f, 0.09851f, 2.85f, 0.009332f, 0.8344f, 0.0f}, {1.026f, 0.1439f, 3.9f, 0.1786f, 0.8164f, 0.04263f},
     {1.762f, 0.1987f, 4.39f, 0.2438f, 0.6367f, 0.09061f}},
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
