"""The transform launcher refuses a pass that is not built (host code, no GPU): the forward pass
that writes the residual has no kernel for radices above 16, alone and for several slices.  Without
that check another operator would run in its place."""
import os
import subprocess

from paper_2008_09042_amd import _lib

PKG = os.path.dirname(_lib.LIB_PATH)
PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include "common.h"
using namespace mx;
int main() {
  FftLaunch l;
  std::memset(&l, 0, sizeof(l));
  l.variant = 9;
  l.blocks = 1;
  l.threads = 64;
  FftMulti m;
  std::memset(&m, 0, sizeof(m));
  m.n = 1;
  m.start[1] = 1;
  std::printf("%d %d %d\n", (int)fft_tr32_launch(l, nullptr), (int)fft_tr32_multi(9, 64, 0, m, nullptr),
              (int)hipErrorInvalidValue);
}
"""


def test_unbuilt_pass_is_an_error(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(PKG, "csrc"),
                    str(src), _lib.LIB_PATH, "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath," + PKG, "-Wl,-rpath,/opt/rocm/lib",
                    "-o", str(exe)], check=True)
    # no GPU is shown to it: a launch, were one tried, could not run
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", ROCR_VISIBLE_DEVICES="-1")
    one, many, invalid = subprocess.run([str(exe)], check=True, capture_output=True, text=True, env=env,
                                        timeout=60).stdout.split()
    assert one == invalid and many == invalid, (one, many, invalid)
