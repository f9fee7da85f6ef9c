// Offsets of the direct loads of operand tiles that may end before the tile does, and the choice
// of a GEMM's tile: plain arithmetic, usable (and tested) on the host as well.
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#define TMZ_HD __host__ __device__ __forceinline__
#else
#define TMZ_HD inline
#endif

namespace tmz {

// A tile of 256 bf16 rows of d values, BK columns per stage, loaded by the waves of a block of
// NT threads: a load is 64 chunks of 16 bytes, kRows whole stage rows.  Load j of wave w takes
// rows (w * kPerWave + j) * kRows .. + kRows - 1; chunk c of row r sits at LDS chunk c ^ swz(r).
//   A load's address is the buffer's base + lane_off + step_off.  The whole row is in the
// per-lane part, which is what a buffer's range check is sure to cover: a row past the end of
// the buffer is out of range by lane_off alone.  The wave-uniform part only moves along the
// row, so it is less than any buffer of at least one row.
template <int BK, int NT>
struct RowLoads {
  static constexpr int kRowB = 2 * BK;                 // bytes per stage row
  static constexpr int kChunks = kRowB / 16;           // 16-byte chunks per stage row
  static constexpr int kRows = 64 / kChunks;           // rows per load
  static constexpr int kPerWave = 256 * kChunks / NT;  // loads per wave per stage
  static_assert(kChunks == 8 || kChunks == 4, "stage width");
  static TMZ_HD int swz(int row) { return kChunks == 8 ? ((row >> 1) & 7) : ((row >> 2) & 3); }
  static TMZ_HD int row(int wave, int j, int lane) {
    return (wave * kPerWave + j) * kRows + lane / kChunks;
  }
  static TMZ_HD uint32_t lane_off(int wave, int j, int lane, int64_t d) {
    const int r = row(wave, j, lane);
    return (uint32_t)(r * d * 2) + 16u * (uint32_t)((lane % kChunks) ^ swz(r));
  }
  static TMZ_HD uint32_t step_off(int kt) { return (uint32_t)kt * kRowB; }
};

// The tiles of the int8 GEMM on shapes that do not fill the compute units with whole 256 x 256
// tiles, and what a launch of T of them takes on cu compute units (us): the first tile of a compute
// unit c0 + l K, further ones a + b K each.  Where T is not a multiple of cu the last, partial
// round counts half of its share and half of a whole one (several blocks share a compute unit).
// Fitted to the nine widths of the decoders at 256 to 8192 tokens, each mode and type by itself
// (rms 3 to 7%): a residual output reads what it adds to, which costs most in the small fp32
// tiles.  The tile with the least estimate is taken: over those shapes within 1% of the best one
// on average, 11% at worst.
enum GemmTile { kTile64, kTile128, kTile256, kTileHalf, kGemmTiles };   // half: whole tiles only
enum GemmKind { kStoreBf16, kStoreF32, kResidualBf16, kResidualF32, kSwiGLU, kGemmKinds };
struct TileCost {
  int bm, bn;
  float c0, l, a, b;                   // l and b in us per 1000 of K; bm 0: not built
};
// kTile64: 64 x 64, for the gate|up product 64 x 128.  kTile256: 128 x 256 with predicated edges;
// not for residual outputs, where it has no registers for the values it adds to (bf16 it spilled
// 73 and 4096 x 1536 -> 1536 took 27.4 us, 16.4 as 128 x 128; fp32 105, 48.1 and 21.5).
// kTileHalf: the same 128 x 256 without edges, for M % 128 = N % 256 = 0.
constexpr TileCost kTileCosts[kGemmKinds][kGemmTiles] = {
    {{64, 64, 3.94f, 1.60f, 0.55f, 0.97f}, {128, 128, 5.38f, 3.06f, 2.00f, 2.95f},
     {128, 256, 7.11f, 5.52f, 3.37f, 5.60f}, {128, 256, 6.86f, 6.03f, 2.98f, 5.53f}},
    {{64, 64, 4.71f, 1.64f, 0.88f, 0.94f}, {128, 128, 6.80f, 3.13f, 3.55f, 2.84f},
     {128, 256, 10.31f, 5.63f, 6.97f, 5.42f}, {128, 256, 8.17f, 6.05f, 4.34f, 5.39f}},
    {{64, 64, 4.66f, 1.59f, 0.66f, 1.03f}, {128, 128, 5.82f, 3.19f, 3.35f, 2.98f},
     {0, 0, 0.f, 0.f, 0.f, 0.f}, {128, 256, 7.88f, 6.12f, 5.63f, 5.31f}},
    {{64, 64, 5.55f, 1.72f, 1.70f, 0.94f}, {128, 128, 7.78f, 3.39f, 6.80f, 2.70f},
     {0, 0, 0.f, 0.f, 0.f, 0.f}, {128, 256, 8.67f, 6.36f, 9.90f, 4.73f}},
    {{64, 128, 4.90f, 1.91f, 0.55f, 1.79f}, {0, 0, 0.f, 0.f, 0.f, 0.f},
     {128, 256, 6.91f, 5.38f, 1.58f, 5.85f}, {128, 256, 7.07f, 5.81f, 1.30f, 5.89f}}};

inline float tile_cost(const TileCost& t, int64_t M, int64_t K, int64_t N, int cu) {
  const int64_t T = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
  const float k = 1e-3f * (float)K, r = (float)T / (float)cu;
  const float more = 0.5f * (float)((T + cu - 1) / cu - 1) + (r > 1.0f ? 0.5f * (r - 1.0f) : 0.0f);
  return t.c0 + t.l * k + more * (t.a + t.b * k);
}
// whole: the tile without edges may be taken.
inline GemmTile choose_tile(GemmKind kind, int64_t M, int64_t K, int64_t N, bool whole, int cu) {
  GemmTile best = kTile64;
  float least = tile_cost(kTileCosts[kind][kTile64], M, K, N, cu);
  for (int t = kTile128; t <= (whole ? kTileHalf : kTile256); ++t) {
    if (kTileCosts[kind][t].bm == 0) continue;
    const float c = tile_cost(kTileCosts[kind][t], M, K, N, cu);
    if (c <= least) {
      least = c;
      best = (GemmTile)t;
    }
  }
  return best;
}

}  // namespace tmz
