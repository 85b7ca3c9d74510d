"""How the 3x3 weight gradient of image tiles is split (patch_wgrad_plan in conv.h), compiled for the host: the room of the partial
results is kept to, no sum counts more rounding than by either kernel in its longest chains, and filter rows are taken only where no CU gets
much more to do than with nine taps, or nine taps cannot be as near."""
import subprocess

from paper_2509_23241_amd import build

PROGRAM = r"""
#include <cstdio>
#include "conv.h"
int main() {
  long rows = 0, nine = 0;
  for (int ci = 1; ci <= 16; ++ci)
    for (int co = 1; co <= 16; ++co)
      for (long px = 1; px <= 5000; px += px < 70 ? 1 : px / 23) {
        const tp::PatchWgradPlan p = tp::patch_wgrad_plan(px, 64 * ci, 64 * co);
        auto most = [](long a, long b) { return (a + b - 1) / b; };
        const long blocks = ci * co, ranges = 256 / blocks > px ? px : 256 / blocks > 1 ? 256 / blocks : 1, tiles = most(px, ranges);
        const long own = most(px, p.splits);
        const long rows_of = 256 / (3 * blocks) > px ? px : 256 / (3 * blocks) > 1 ? 256 / (3 * blocks) : 1, row_tiles = most(px, rows_of);
        const double by_eights = 34 + (row_tiles + 7) / 8 + rows_of / 10., all = 8. * px / ranges;
        bool ok = p.splits >= 1 && p.splits <= ranges && p.apart >= 1;
        if (p.rows) {
          bool nine_near = false;
          for (long a = 1; a <= 64 && a <= tiles; ++a) nine_near = nine_near || 8 * a + most(tiles, a) + 1 + ranges / 10. <= by_eights;
          ok = ok && p.splits == rows_of && p.apart <= 8 && 4 * p.apart + most(own, p.apart) + 2 + rows_of / 10. < all + ranges / 10.;
          ok = ok && (px >= 2 * ranges || own == 1);
          ok = ok && (!nine_near || 3 * own * most(3 * blocks * rows_of, 256) <= 1.6 * 9 * tiles + 3);
        } else {
          ok = ok && p.splits == ranges && 8 * p.apart + most(own, p.apart) + 1 + ranges / 10. <= by_eights + 1e-9;
        }
        if (!ok) { printf("%d -> %d channels, %ld tiles: %d %d %d\n", 64 * ci, 64 * co, px, p.rows, p.splits, p.apart); return 1; }
        ++(p.rows ? rows : nine);
      }
  printf("%ld by rows, %ld with nine taps\n", rows, nine);
  return rows && nine ? 0 : 1;
}
"""


def test_plan_of_patch_weight_gradients(tmp_path):
    source, program = tmp_path / "plan.hip", tmp_path / "plan"
    source.write_text(PROGRAM)
    subprocess.run([build._hipcc(), "--offload-host-only", "-std=c++17", "-O1", "-I", build.CSRC, "-x", "hip", str(source), "-o", str(program)],
                   check=True, capture_output=True)
    run = subprocess.run([str(program)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout
