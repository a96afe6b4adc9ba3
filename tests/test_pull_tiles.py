"""CPU check of the rule for pull tiles (pull_tile_words), compiled for the host."""
import os
import subprocess

from paper_1804_03327_amd import build

HARNESS = r"""
#include "dobfs_internal.h"
#include <cstdio>
using namespace dobfs;
int main() {
  const int64_t mosts[] = {1, 16, 768, kExpandBlocks};
  for (int64_t most : mosts)
    for (int64_t n = 1; n < 300000; n = n < 3000 ? n + 1 : n + 509) {
      const int32_t w = pull_tile_words(n, most);
      const int64_t tiles = (n + w - 1) / w;
      const bool size = w >= kPullTileMin && w <= kPullTileWords && w % kPullTileMin == 0;
      const bool fits = tiles <= most || w == kPullTileWords;          // no more tiles than blocks
      const bool small = w == kPullTileMin || (n + w / 2 - 1) / (w / 2) > most;  // and no larger than that takes
      if (!size || !fits || !small) {
        std::printf("%lld words, %lld blocks: %d\n", (long long)n, (long long)most, w);
        return 1;
      }
    }
  return pull_tile_words(8192) == 8 && pull_tile_words(8192, 768) == 16 ? 0 : 2;
}
"""


def test_pull_tiles_fit_the_blocks(tmp_path):
    src = tmp_path / "h.hip"
    src.write_text(HARNESS)
    exe = str(tmp_path / "h")
    subprocess.run([build.HIPCC, "--offload-arch=" + build.ARCH, "-std=c++17", "-I" + build.CSRC,
                    "-I" + os.path.join(build.ROOT, "include"), str(src), "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
