"""The deal of point blocks to the tiles of the FP32 and FP64 sweeps (csrc/sweep_tiles.h), on the host:
every block in exactly one tile, and a kernel for every tile's count, for both kinds of addressing.
Five FP64 blocks (65 to 80 points) in tiles of a fixed four gave a block to two tiles, whose
workgroups both added into its rows."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1504_07690_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "sweep_tiles.h"
int main() {
  long cases = 0;
  for (int max_mb : {2, 4})  // FP32, FP64
    for (int wide = 0; wide < 2; ++wide)
      for (long strips : {1L, 7L, 300L, 5000L, 1L << 21})
        for (int nb = 1; nb <= 4096; nb += (nb < 600 ? 1 : 37)) {
          const ssm::SweepTiling t = ssm::sweep_tiling(strips, nb, max_mb, wide);
          const int mb = t.mb();
          bool ok = t.nb == nb && t.mt >= 1 && mb >= 1 && mb <= max_mb;
          std::vector<int> owners(nb, 0);
          for (int m = 0; ok && m < t.mt; ++m) {
            const int strip = mb == 1 || t.count(m) == mb ? mb : mb - 1;  // what the kernel runs
            ok = t.count(m) == strip;
            for (int b = t.first(m); b < t.first(m) + strip && b < nb; ++b) ++owners[b];
          }
          for (int o : owners) ok = ok && o == 1;
          if (!ok) {
            std::printf("max_mb %d wide %d strips %ld nb %d: mt %d mb %d\n", max_mb, wide, strips, nb, t.mt, mb);
            return 1;
          }
          ++cases;
        }
  std::printf("%ld\n", cases);
}
"""


def test_every_block_has_one_tile(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++") or shutil.which("amdclang++")
    if cxx is None:
        pytest.skip("no host compiler")
    src = tmp_path / "tiling.cpp"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(tmp_path / "tiling")], check=True)
    res = subprocess.run([str(tmp_path / "tiling")], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
    assert int(res.stdout) > 10000
