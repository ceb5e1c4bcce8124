"""The arithmetic of the one-pass scan at the largest counts it takes, on the CPU: tiles of n cells, and the
cell numbers of the last tile, against 64-bit arithmetic up to n = 2^31 - 1 (compiled from the header
that the kernels and the launches use)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "pcol_internal.h"
#include <cstdio>
int main() {
  using namespace pcol;
  const int64_t top = 2147483647;
  const int64_t ns[] = {1,       SCAN_B - 1,       SCAN_B,       SCAN_B + 1,       1 << 28,  top - 2 * SCAN_B,
                        top - SCAN_B, top - SCAN_B + 1, top - SCAN_B + 2, 2147483000, top - 1, top};
  for (int64_t n : ns) {
    const int64_t want = n / SCAN_B + (n % SCAN_B ? 1 : 0);
    // the last cell number that the last tile's last thread forms, in range or not
    const int64_t last = (want - 1) * SCAN_B + (int64_t)(SCAN_T - 1) * SCAN_E + SCAN_E - 1;
    if (scan_tiles(n) != want || last > top || want * SCAN_B < n) {
      std::printf("n %lld: %d tiles, not %lld; last cell %lld\n", (long long)n, scan_tiles(n),
                  (long long)want, (long long)last);
      return 1;
    }
  }
  return 0;
}
"""


def test_tiles_up_to_the_largest_count(tmp_path):
    src, exe = tmp_path / "tiles.hip", tmp_path / "tiles"
    src.write_text(SOURCE)
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-std=c++17", "-O1", "-Xclang", "-target-feature",
                           "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
                           "-I", os.path.join(ROOT, "paper_2501_05340_amd", "csrc"), str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout + out.stderr
