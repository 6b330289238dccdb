"""The step's workspace layout (no GPU): its constexpr layout function is
evaluated by the compiler, so nothing here is a second copy of it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_06557_amd", "csrc")

CHECK = """
#include "cascade_step.hip"
namespace cascade {
namespace {
// The tiled sort stores splitters while other workgroups of the launch read
// eval's partials, so its words must end where the partials begin; eval's
// clear ends where the samples begin.
constexpr bool apart(int n) {
  const Layout L = make_layout(n);
  return L.tiles <= kTiledTiles && (long long)L.tile * L.tiles >= n &&
         L.samples >= L.sort_status &&
         L.splitters >= L.samples + (size_t)L.tiles * samples_of(L.tile) * 8 &&
         L.tiled_end >= L.splitters + (size_t)L.tiles * 8 && L.tiled_end <= L.partials;
}
constexpr bool all_apart(int from, int to, int by) {
  for (int n = from; n <= to && n <= kTiledMax; n += by)
    for (int d = 0; d < 2; ++d)
      if (n + d <= kTiledMax && !apart(n + d)) return false;
  return true;
}
static_assert(all_apart(kSmallMax + 1, 9000, 1), "every small queue");
static_assert(all_apart(9216, kTiledMax, 256), "both sides of every tile");
// a workspace for n requests serves every smaller queue
constexpr bool grows(int to, int by) {
  for (int n = 1; n < to; n += by)
    if (make_layout(n).total > make_layout(n + 1).total ||
        make_layout(n).total > make_layout(n + by).total)
      return false;
  return true;
}
static_assert(grows(3000, 1) && grows((1 << 20) - 256, 255), "monotone");
}  // namespace
}  // namespace cascade
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not installed")
def test_tiled_sort_words_stay_clear_of_the_partials(tmp_path):
    src = tmp_path / "layout.hip"
    src.write_text(CHECK)
    out = subprocess.run(["hipcc", "-x", "hip", "--cuda-host-only", "-fsyntax-only", "-std=c++17",
                          "-fconstexpr-steps=200000000", "-I", os.path.join(ROOT, "include"),
                          "-I", CSRC, str(src)], capture_output=True, text=True, timeout=600)
    assert out.returncode == 0, out.stderr[-3000:]
