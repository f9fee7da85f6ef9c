"""Address arithmetic of the direct loads of partial tiles, on the host: whatever part of the
offset a buffer's range check looks at, a row past the end must be out of range by the per-lane
part alone, and the scalar part must not lead a row in range out of it."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "tmz_tiles.h"
template <int BK, int NT> long long check(long long d, int rows) {
  using L = tmz::RowLoads<BK, NT>;
  const unsigned long long bytes = (unsigned long long)rows * d * 2;   // the buffer of the tile
  long long bad = 0;
  bool seen[256][L::kChunks] = {};
  for (int w = 0; w < NT / 64; ++w)
    for (int j = 0; j < L::kPerWave; ++j)
      for (int lane = 0; lane < 64; ++lane) {
        const int r = L::row(w, j, lane);
        const unsigned long long v = L::lane_off(w, j, lane, d);
        const int c = (lane % L::kChunks) ^ L::swz(r);
        bad += r < 0 || r >= 256 || seen[r][c];
        seen[r][c] = true;
        if (r >= rows) { bad += v < bytes; continue; }                 // fetches nothing
        for (int kt = 0; kt < d / BK; ++kt) {
          const unsigned long long s = L::step_off(kt);
          bad += s >= bytes || v + s + 16 > bytes;
          bad += v + s != (unsigned long long)r * d * 2 + 2ull * BK * kt + 16 * c;
        }
      }
  return bad;
}
int main() {
  long long bad = 0;
  for (long long d : {64ll, 192ll, 256ll, 1536ll, 2560ll, 8192ll})
    for (int rows : {1, 2, 3, 7, 8, 9, 15, 16, 17, 31, 32, 33, 128, 203, 255, 256}) {
      const long long b = check<64, 512>(d, rows);
      if (b) printf("d %lld rows %d: %lld\n", d, rows, b);
      bad += b;
    }
  bad += check<32, 512>(96, 5) + check<64, 256>(128, 19);
  return bad != 0;
}
"""


def test_rows_past_the_end_are_out_of_range_by_the_lane_offset(tmp_path):
    src = tmp_path / "loads.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "loads")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2609_33548_amd", "csrc"),
                    str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
