// Offsets of the direct loads of operand tiles that may end before the tile does: plain
// integer arithmetic, usable (and tested) on the host as well.
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

}  // namespace tmz
