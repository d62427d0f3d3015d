"""The grid of the tile path's middle-pass kernel, whose workgroups wait for one
another: never more than the device holds at once. Host code of the library's
own header, compiled with the host compiler; no GPU."""

import os
import shutil
import subprocess

import pytest

from tests._lib import ROOT

HIP = "/opt/rocm/include"

PROGRAM = r"""
#include <cstdio>
#include "kernels.h"
int main() {
  const long long sizes[] = {16385, 65536, 131073, 1 << 20, (1 << 20) + 1, 1 << 21};
  for (long long n : sizes)
    for (int resident : {1, 20, 32, 64, 100, 128, 256, 512})
      for (long long tile : {1024, 2048, 4096, 8192}) {
        const long long tiles = (n + tile - 1) / tile;
        const int g = semsched::tile_mid_groups(n, tiles, resident);
        if (g < 1 || g > resident || g > tiles || g > (n <= 1 << 20 ? 64 : 128)) {
          std::printf("n=%lld tiles=%lld resident=%d: %d\n", n, tiles, resident, g);
          return 1;
        }
      }
  // a whole device takes what it took
  return semsched::tile_mid_groups(1 << 20, 128, 256) == 64 &&
                 semsched::tile_mid_groups(1 << 21, 256, 256) == 128 &&
                 semsched::tile_mid_groups(20000, 20, 512) == 20
             ? 0
             : 2;
}
"""


@pytest.mark.skipif(not (shutil.which("g++") and os.path.isdir(HIP)), reason="needs g++ and HIP")
def test_grid_fits_the_device(tmp_path):
    src = tmp_path / "grid.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "grid")
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", HIP, "-I",
                           os.path.join(ROOT, "paper_2506_12204_amd", "csrc"), str(src), "-o", exe])
    subprocess.check_call([exe])
