"""The choice of a GEMM's tile below one round of whole 256 x 256 tiles, on the host: on shapes over
its whole range the chosen tile's measured time is near the best one's, and never above that of
the 128 x 256 tiles without edges (kTileHalf) by more than the measurements differ."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# kind, M, K, N, then us per launch as kTile64, kTile128, kTile256, kTileHalf (0: not built),
# MI355X, the operands in the caches
MEASURED = [
    ("kResidualBf16", 256, 1536, 1536, 7.0, 10.3, 0, 16.9),
    ("kResidualBf16", 4096, 1536, 1536, 18.0, 16.4, 0, 18.7),
    ("kResidualBf16", 8192, 1536, 1536, 33.0, 26.2, 0, 27.3),
    ("kResidualBf16", 3072, 4096, 1536, 30.4, 29.5, 0, 33.3),
    ("kResidualBf16", 2048, 2560, 2560, 21.5, 21.5, 0, 24.6),
    ("kResidualBf16", 6144, 2560, 2560, 55.4, 43.7, 0, 39.7),
    ("kResidualBf16", 4096, 6912, 2560, 84.7, 70.9, 0, 79.9),
    ("kResidualBf16", 6144, 6912, 2560, 124.8, 95.1, 0, 86.4),
    ("kResidualF32", 4096, 1536, 1536, 25.0, 21.5, 0, 21.8),
    ("kResidualF32", 8192, 1536, 1536, 42.2, 34.3, 0, 30.5),
    ("kResidualF32", 4096, 4096, 1536, 38.6, 35.6, 0, 37.0),
    ("kResidualF32", 1536, 2560, 2560, 21.6, 19.5, 0, 26.4),
    ("kResidualF32", 3072, 2560, 2560, 36.8, 29.1, 0, 29.7),
    ("kResidualF32", 6144, 2560, 2560, 64.8, 53.4, 0, 44.0),
    ("kResidualF32", 2560, 6912, 2560, 64.3, 50.5, 0, 52.6),
    ("kResidualF32", 8192, 256, 256, 8.0, 9.4, 0, 11.0),
    ("kStoreBf16", 256, 2560, 2560, 8.0, 12.2, 20.1, 21.2),
    ("kStoreBf16", 4096, 1536, 1536, 16.3, 15.1, 16.6, 17.1),
    ("kStoreBf16", 2048, 2560, 6912, 46.7, 38.8, 35.7, 36.1),
    ("kStoreBf16", 6144, 6912, 2560, 120.4, 92.1, 84.0, 84.5),
    ("kStoreF32", 3072, 1536, 4608, 35.8, 32.4, 31.4, 27.9),
    ("kStoreF32", 512, 2560, 3840, 11.5, 14.2, 23.8, 22.6),
    ("kStoreF32", 6144, 2560, 2560, 54.7, 45.0, 43.7, 39.4),
    ("kStoreF32", 2048, 2560, 6912, 50.4, 42.9, 41.9, 38.4),
    ("kSwiGLU", 256, 1536, 8192, 8.1, 0, 14.2, 14.9),
    ("kSwiGLU", 1024, 2560, 13824, 39.5, 0, 34.2, 35.0),
]

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "tmz_tiles.h"
int main(int argc, char** argv) {
  for (int i = 1; i + 3 < argc; i += 4)
    std::printf("%d %d\n",
                tmz::choose_tile((tmz::GemmKind)std::atoi(argv[i]), std::atoll(argv[i + 1]),
                                 std::atoll(argv[i + 2]), std::atoll(argv[i + 3]), true, 256),
                tmz::choose_tile((tmz::GemmKind)std::atoi(argv[i]), std::atoll(argv[i + 1]),
                                 std::atoll(argv[i + 2]), std::atoll(argv[i + 3]), false, 256));
}
"""


def test_chosen_tiles_are_near_the_best(tmp_path):
    src = tmp_path / "choice.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "choice")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2609_33548_amd", "csrc"),
                    str(src), "-o", exe], check=True)
    kinds = ["kStoreBf16", "kStoreF32", "kResidualBf16", "kResidualF32", "kSwiGLU"]
    args = [str(v) for r in MEASURED for v in (kinds.index(r[0]), *r[1:4])]
    out = subprocess.run([exe, *args], capture_output=True, text=True, check=True).stdout.split()
    for r, whole, ragged in zip(MEASURED, out[::2], out[1::2]):
        us = r[4:]
        built = [t for t in us if t > 0]
        assert us[int(whole)] > 0 and us[int(whole)] <= 1.12 * min(built), r
        assert us[int(whole)] <= 1.03 * us[3], r
        assert int(ragged) < 3 and us[int(ragged)] > 0
        assert us[int(ragged)] <= 1.12 * min(t for t in us[:3] if t > 0), r
