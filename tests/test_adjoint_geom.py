"""The split of the dense adjoint into workgroups (host code, no GPU): the library's own rule,
compiled from its header.  Every row, column group and coil is covered, no more row chunks than
asked for, and where the rows are many the workgroups fill the rounds over the compute units."""
import itertools
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2008_09042_amd", "csrc")
PROGRAM = r"""
#include <cstdio>
#include "adjoint_geom.h"
int main() {
  long long N, K;
  int J, m;
  while (std::scanf("%lld %lld %d %d", &N, &K, &J, &m) == 4) {
    const mx::AdjGeom a = mx::adj_geom(N, K, J, m);
    std::printf("%d %d %d %d %d %lld %d\n", a.JB, a.AKB, a.jgs, a.kwl, a.ks, (long long)a.chunk, a.nchunk);
  }
}
"""


@pytest.fixture(scope="module")
def geom(tmp_path_factory):
    d = tmp_path_factory.mktemp("geom")
    (d / "t.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + CSRC, str(d / "t.cpp"), "-o", str(d / "t")], check=True)

    def run(cases):
        text = "".join("%d %d %d %d\n" % c for c in cases)
        out = subprocess.run([str(d / "t")], input=text, check=True, capture_output=True, text=True).stdout.split("\n")
        return [tuple(int(v) for v in line.split()) for line in out if line]

    return run


def test_every_block_is_covered(geom):
    cases = list(itertools.product((1, 15, 16, 127, 128, 4096, 131071, 131072, 10 ** 6), (1, 32, 33, 64, 65, 128, 129, 256, 257, 600, 5000),
                                   (1, 16, 17, 32, 33, 64, 65, 200, 1000), (0, 1, 7)))
    for (N, K, J, m), (JB, AKB, jgs, kwl, ks, chunk, nchunk) in zip(cases, geom(cases)):
        step = 16 * (8 >> kwl)
        assert chunk % step == 0 and (nchunk - 1) * chunk < N <= nchunk * chunk
        assert 0 < nchunk and (m == 0 or nchunk <= m)
        assert jgs * JB * 16 >= J and ks * (AKB << kwl) * 16 >= K
        assert 2 ** kwl * JB * AKB * 2 * 64 * 16 * ((8 >> kwl) // 2) <= 160 * 1024  # the row groups' tiles in LDS


def test_rounds_are_full(geom):
    """N of whole steps in plenty: at most a tenth of the last round over 256 compute units is idle
    (two workgroups to a unit up to 16 coils)."""
    N = 10 ** 7
    cases = [(N, K, J, 0) for K in range(20, 4000, 61) for J in (3, 16, 20, 32, 33, 64, 100, 200, 400)]
    for (_, K, J, _), (JB, AKB, jgs, kwl, ks, chunk, nchunk) in zip(cases, geom(cases)):
        slots = 512 if JB == 1 else 256
        n = nchunk * jgs * ks
        assert n >= 0.89 * (-(-n // slots) * slots), (K, J, n)  # a chunk rounds up to whole steps: 1 % less
