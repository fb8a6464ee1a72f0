"""Where a lane of a wave's own tile copy (WaveDma) reads, compiled for the host, against the layout of a tile in LDS: row strides
that are odd multiples of 16 bytes among them, full tiles and tiles with fewer rows, all passes of a tile and one at a time."""
import subprocess

from paper_2504_14519_amd.build import CSRC, HIPCC

PROGRAM = r"""
#include <stdio.h>
#include "tile_common.hpp"
using namespace slimpipe;

// lanes whose source is not what the layout puts at their place
template <int D, int ROWS>
static void check(int64_t stride) {
  using W = WaveDma<D, ROWS>;
  const uint32_t row_bytes = (uint32_t)stride * 2;
  int full = 0, clamped = 0, alone = 0;
  for (int row = 0; row < ROWS; ++row)
    for (int chunk = 0; chunk < D / 8; ++chunk) {
      const int place = tile_off<D>(row, chunk), n = place / 1024, lane = place % 1024 / 16;
      W w;
      w.init(lane, row_bytes);
      full += (int64_t)w.off[n % W::PHASES] + (int64_t)n * W::RPP * row_bytes != (int64_t)row * row_bytes + chunk * 16;
      for (int rows : {1, 2, ROWS / 2 + 1, ROWS - 1, ROWS}) {
        const int64_t want = (int64_t)(row < rows ? row : rows - 1) * row_bytes + chunk * 16;
        alone += (int64_t)W::pass_off(lane, n, row_bytes, rows) != want;
        for (int first : {-5, 0, 1, rows - 1}) {
          const int r = row < first ? first : row;
          if (first < rows) clamped += (int64_t)w.clamped(lane, n, row_bytes, first, rows) != (int64_t)(r < rows ? r : rows - 1) * row_bytes + chunk * 16;
        }
      }
    }
  if (full || clamped || alone) printf("D %d rows %d stride %d: full %d clamped %d alone %d\n", D, ROWS, (int)stride, full, clamped, alone);
}

int main() {
  for (int64_t stride : {64, 72, 80, 128, 136, 144, 152, 264, 1024, 1032, 1040, (1 << 22) - 8}) {
    check<64, 32>(stride);
    check<64, 64>(stride);
    if (stride >= 128) check<128, 32>(stride);
  }
  printf("done\n");
  return 0;
}
"""


def test_wave_copy_reads_the_rows_of_its_tile(tmp_path):
    src, exe = str(tmp_path / "copy.hip"), str(tmp_path / "copy")
    with open(src, "w") as f:
        f.write(PROGRAM)
    r = subprocess.run([HIPCC, "--offload-host-only", "-O2", "-std=c++17", "-w", "-I", CSRC, src, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0
    assert r.stdout == "done\n"
