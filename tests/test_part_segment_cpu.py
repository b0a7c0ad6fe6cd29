"""The one-segment lookup of launches with a whole number of work-groups per query tile, and the
merge's owner rule for them, against the general split arithmetic (both compiled from
csrc/seg_table.hpp with the host compiler), over every part count and a range of tile counts up
to the largest a cache allows."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include <initializer_list>
#include "seg_table.hpp"
using namespace unstep;
int main() {
  const int32_t tks[] = {1, 2, 3, 4, 5, 7, 8, 19, 52, 71, 255, 256, 257, 293, 400, 4095, 65537, 131072};
  long n = 0;
  for (int32_t Tk : tks)
    for (int32_t parts = 1; parts <= 256 && parts <= Tk; ++parts)
      for (int32_t tiles : {1, 2, 3, 7, 84, 228, 8388607}) {
        if ((parts > 1 && int64_t(tiles) * parts > 256) || int64_t(tiles) * Tk > (int64_t(1) << 35)) continue;
        Schedule sc;
        sc.Tk = Tk;
        sc.U = int64_t(tiles) * Tk;
        sc.G = int64_t(tiles) * parts;
        const int32_t step = tiles > 1000 ? 524287 : 1;
        for (int64_t g = 0; g < sc.G; g += step, ++n) {
          const int64_t lo = sc.start(g);
          int64_t hi = sc.start(g + 1);
          const Segment a = take_segment(sc, lo, hi), b = part_segment(Tk, parts, int32_t(g));
          if (hi != lo || a.t != b.t || a.k0 != b.k0 || a.k1 != b.k1 || a.slot != b.slot || a.full != b.full || b.k0 >= b.k1) {
            std::printf("Tk %d parts %d tiles %d g %lld\n", Tk, parts, tiles, (long long)g);
            return 1;
          }
          const int64_t ua = b.t * Tk;               // the merge: owners t parts .. t parts + parts - 1, all in slot 0
          if (sc.owner(ua) != b.t * parts || sc.owner(ua + Tk - 1) != b.t * parts + parts - 1 || sc.start(b.t * parts) < ua) return 2;
        }
      }
  std::printf("ok %ld\n", n);
  return n > 100000 ? 0 : 3;
}
"""


def test_part_segment_equals_the_general_split(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(SOURCE)
    b = subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Wno-unknown-pragmas", "-Werror", f"-I{ROOT}/include",
                        f"-I{ROOT}/paper_2609_32518_amd/csrc", str(src), "-o", str(exe)], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
