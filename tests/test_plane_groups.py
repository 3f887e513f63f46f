"""Launch geometry of the fused plane kernels (host code, no GPU): the library's own choice of coils
per workgroup, compiled from its header, with the index arithmetic of the kernels restated.  Every
(plane, group) pair is visited once, every block that a group reads or writes lies in the buffer
that the plan sizes for it (the gx partials by the adjoint's groups alone), and the image of a
Jacobian product's direction, which takes the gx partials' place, fits there."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2008_09042_amd", "csrc")
PROGRAM = r"""
#include <cstdio>
#include "plane_groups.h"
int main() {
  long long planes;
  int J, cus;
  while (std::scanf("%lld %d %d", &planes, &J, &cus) == 3) {
    const mx::PlaneGroups g = mx::plane_groups(planes, J, cus);
    std::printf("%d %d\n", g.fwd, g.adj);
  }
}
"""
NXCD = 8


@pytest.fixture(scope="module")
def groups(tmp_path_factory):
    """(planes, coils, compute units) -> coils per workgroup (forward, adjoint), many at a time."""
    d = tmp_path_factory.mktemp("groups")
    (d / "t.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + CSRC, str(d / "t.cpp"), "-o", str(d / "t")], check=True)

    def run(cases):
        text = "".join("%d %d %d\n" % c for c in cases)
        out = subprocess.run([str(d / "t")], input=text, check=True, capture_output=True, text=True).stdout.split()
        return [(int(out[2 * i]), int(out[2 * i + 1])) for i in range(len(cases))]

    return run


def plane_block(ngrp, n2):
    nb = ngrp * n2
    l = np.arange(nb)
    if nb % NXCD == 0:
        l = (l % NXCD) * (nb // NXCD) + l // NXCD
    return l // ngrp, l % ngrp


def test_known_choices(groups):
    # 128 planes and 32 coils; 3 coils where halving took 2; forward and adjoint apart
    assert groups([(128, 32, 256), (64, 12, 256), (64, 5, 256), (90, 16, 256)]) == [(16, 16), (3, 3), (2, 2), (2, 8)]


def test_blocks_stay_in_their_buffers(groups):
    planes = [2, 4, 10, 12, 16, 20, 48, 64, 90, 100, 128, 162, 250, 256]
    coils = [1, 2, 3, 5, 6, 7, 8, 12, 16, 17, 20, 31, 32, 48, 64]
    cases = [(n2, J, cus) for n2 in planes for J in coils for cus in (256, 304)]
    some_odd = some_apart = False
    for (n2, J, cus), (fwd, adj) in zip(cases, groups(cases)):
        partials = -(-J // adj)  # of N points each
        assert 1 <= fwd <= 16 and 1 <= adj <= 16
        some_odd |= any(g & (g - 1) for g in (fwd, adj))
        some_apart |= fwd != adj
        for G in (fwd, adj):
            ngrp = -(-J // G)
            i2, gi = plane_block(ngrp, n2)
            assert np.array_equal(np.sort(i2 * ngrp + gi), np.arange(ngrp * n2))
            assert i2.min() >= 0 and i2.max() < n2 and gi.max() < ngrp
            j0, j1 = gi * G, np.minimum(J, (gi + 1) * G)
            assert (j0 < j1).all()  # no empty group; T3, Z blocks (j n2 + i2) below J n2
            assert ((j1 - 1) * n2 + i2).max() < J * n2
            if G == adj and ngrp == partials:
                assert (gi * n2 + i2).max() < partials * n2  # planes of the gx partials
        assert n2 <= partials * n2  # the direction's image, n2 planes
    assert some_odd and some_apart
