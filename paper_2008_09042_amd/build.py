"""Build libmaxwell.so (the C-ABI library) in-tree for gfx950 with hipcc.

    python -m paper_2008_09042_amd.build

Every HIP translation unit under csrc/ is compiled to an object under
csrc/_build/ (in parallel) and linked into paper_2008_09042_amd/libmaxwell.so.
"""
import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD_DIR = os.path.join(CSRC, "_build")
LIB = os.path.join(HERE, "libmaxwell.so")
SOURCES = ["api.hip", "plan.hip", "gemm.hip", "fft_tr16.hip", "fft_tr16_grid.hip", "fft_tr16_multi.hip", "fft_tr32.hip",
           "fft_tr32_grid.hip", "fft_tr32_multi.hip", "fft.hip", "elementwise.hip", "nufft.hip", "tucker_fused.hip",
           "core_contract.hip", "mode3.hip", "solver.hip", "admm.hip", "compress.hip", "stream_maps_fp32.hip",
           "stream_maps_bf16.hip", "stream_gx_fp32.hip", "stream_gx_bf16.hip", "stream_adjoint_fp32.hip",
           "stream_adjoint_bf16.hip", "tucker_rows_fp32.hip", "tucker_rows_bf16.hip", "fft_combine.hip", "diag.hip",
           "tune.hip"]
ARCH = "gfx950"
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# Packed FP32 instructions are disabled for all device code.
CFLAGS = ["--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(src):
    obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC] + CFLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    msgs = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                     if "not a recognized feature for this target" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{msgs}")
    return obj, msgs


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    srcs = [s for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        results = list(ex.map(_compile, srcs))
    objs = [o for o, _ in results]
    if verbose:
        for _, m in results:
            if m.strip():
                print(m)
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout + r.stderr)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
