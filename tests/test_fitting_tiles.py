"""The tiles of a 240-wide layer that the wavefronts of the fitting net's
middle kernel read: all inside the weights, the biases and w_out, also where
there are more wavefronts than tiles, and each owned once.  The kernel's own
functions, compiled for the host: what lies past a caller's weights is never
read, which no value the kernel returns could show."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2107_02103_amd", "csrc", "dpc_fit_tiles.h")

# prints, per number of wavefronts: the largest tile read and the owners of each tile
PROGRAM = r"""
#include <cstdio>
#include "%s"
int main() {
  for (int nw = 1; nw <= 32; ++nw) {
    int top = 0, own[kFt] = {};
    for (int wave = 0; wave < nw; ++wave)
      for (int u = 0; u < (kFt + nw - 1) / nw; ++u) {
        const int t = fit_tile(wave, nw, u);
        if (t > top || t < 0) top = t;
        if (fit_owns(wave, nw, u)) ++own[t];
      }
    std::printf("%%d %%d %%d", nw, top, (int)fit_tiles_ok(nw));
    for (int t = 0; t < kFt; ++t) std::printf(" %%d", own[t]);
    std::printf("\n");
  }
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler")
def test_every_tile_exists(tmp_path):
    src = tmp_path / "tiles.cpp"
    src.write_text(PROGRAM % HEADER)
    subprocess.check_call(["g++", "-std=c++17", str(src), "-o", str(tmp_path / "tiles")])
    for line in subprocess.check_output([str(tmp_path / "tiles")], text=True).splitlines():
        nw, top, ok, *own = map(int, line.split())
        assert 0 <= top < 15 and ok == 1 and own == [1] * 15, nw
        # channel 4 (i % 4) + i / 4 of the tile: the last element of W, the biases and w_out it reaches
        assert (16 * top + 15) * 240 + 16 * 14 + 15 < 240 * 240 and 16 * top + 15 < 240
