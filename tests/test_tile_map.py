"""Order of a dense product's output tiles (make_uneven_tile_map in mfma_common.h), compiled for the host: every tile once, and no
XCD's CUs with more rounds of tiles than when the tiles are dealt out evenly."""
import subprocess

from paper_2509_23241_amd import build

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "mfma_common.h"
int main() {
  const int tile[5][2] = {{64, 64}, {128, 64}, {128, 128}, {256, 128}, {256, 256}};
  long uneven = 0;
  for (auto& t : tile)
    for (int m = 1; m <= 140; m += m < 40 ? 1 : 7)
      for (int n = 1; n <= 140; n += n < 40 ? 1 : 7) {
        const tp::TileMap map = tp::make_uneven_tile_map(m, n, t[0], t[1]);
        std::vector<int> seen(m * n), of_xcd(8);
        for (int b = 0; b < map.grid(); ++b) {
          int i, j;
          map.get(b, i, j);
          if (i < 0 || j < 0) { printf("%d x %d: workgroup %d gets tile %d %d\n", m, n, b, i, j); return 1; }
          if (!map.inside(i, j)) continue;
          ++seen[i * n + j];
          ++of_xcd[b & 7];
        }
        for (int k = 0; k < m * n; ++k)
          if (seen[k] != 1) { printf("%d x %d: tile %d %d times\n", m, n, k, seen[k]); return 1; }
        const int even = (m * n + 7) / 8;
        uneven += map.xm && (m % map.xm || n % map.xn);
        for (int k = 0; k < 8; ++k)
          if (map.xm && (of_xcd[k] + 31) / 32 > (even + 31) / 32) {
            printf("%d x %d tiles of %d x %d: %d on one XCD of 32 CUs, %d dealt out evenly\n", m, n, t[0], t[1], of_xcd[k], even);
            return 1;
          }
      }
  printf("%ld uneven\n", uneven);
  return uneven ? 0 : 1;
}
"""


def test_every_tile_once_and_no_cu_with_another_round(tmp_path):
    source, program = tmp_path / "tiles.hip", tmp_path / "tiles"
    source.write_text(PROGRAM)
    subprocess.run([build._hipcc(), "--offload-host-only", "-std=c++17", "-O1", "-I", build.CSRC, "-x", "hip", str(source), "-o", str(program)],
                   check=True, capture_output=True)
    run = subprocess.run([str(program)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout
