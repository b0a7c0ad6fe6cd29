"""The projection's choice of kernel and tile (csrc/linear_plan.hpp, compiled with the host compiler):
which tile each size takes, and that every launch it plans fits 32 bits of work-items, up to the
largest outputs that any of its kernels can take."""
import os
import shutil
import subprocess

import pytest

from tests.test_gpu_linear_exact import SHAPES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include "linear_plan.hpp"
int main() {
  int M, N, K;
  while (std::scanf("%d %d %d", &M, &N, &K) == 3) {
    const unstep::LinearTile t = unstep::linear_plan(M, N, K);
    std::printf("%d %d %d %d %d %d\n", t.bn, t.bm, t.staged, t.tiles_n, t.tiles_m, t.fits);
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("plan")
    (d / "t.cpp").write_text(SOURCE)
    b = subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                        f"-I{ROOT}/paper_2609_32518_amd/csrc", str(d / "t.cpp"), "-o", str(d / "t")], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr

    def ask(shapes):
        r = subprocess.run([str(d / "t")], input="\n".join("%d %d %d" % s for s in shapes), capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        return [tuple(map(int, l.split())) for l in r.stdout.splitlines()]
    return ask


def test_largest_outputs_fit_one_launch(plan):
    """Tall and wide products around every power of two up to INT32_MAX rows or columns."""
    big = [2 ** p + d for p in (20, 23, 26, 28, 29, 30) for d in (-1, 0, 1)] + [2 ** 31 - 2 ** 12, 2 ** 31 - 1]
    shapes = []
    for a in big:
        for b in (8, 64, 72, 128, 136, 1024, 16384):
            shapes += [(a, b, k) for k in (8, 64, 72, 2 ** 22)] + [(b, a // 8 * 8, k) for k in (8, 64, 2 ** 22)]
    for (M, N, K), (bn, bm, staged, tn, tm, fits) in zip(shapes, plan(shapes)):
        assert (tn, tm) == (-(-N // bn), -(-M // bm)), (M, N, K)
        threads = 256 if staged else 512
        small, large = -(-M // 128) * -(-N // 128) * 256, -(-M // 256) * -(-N // 128) * 512
        assert fits == (small < 2 ** 32 or (K < 2 ** 22 and large < 2 ** 32)), (M, N, K)
        if fits:
            assert tn * tm * threads < 2 ** 32, (M, N, K, bn, bm, staged)
    assert plan([(2 ** 30, 8, 8)])[0][5] and plan([(2 ** 30, 64, 40)])[0][5]


def test_tiles_of_the_exact_cases(plan):
    """The sizes that the GPU test of whole numbers names reach every tile and the staged kernel."""
    got = plan([s[:3] for s in SHAPES])
    assert [(bn, bm, bool(staged)) for bn, bm, staged, *_ in got] == [s[3] for s in SHAPES]
    assert {s[3] for s in SHAPES} == {(128, 256, False), (128, 128, False), (64, 128, False), (64, 64, False), (128, 128, True)}
