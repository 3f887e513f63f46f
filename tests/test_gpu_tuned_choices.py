"""The dense basis' plan-time choices: every use with the other uses' opposite choice (given by a
tuning file: a choice is four times the GEMM's split, plus 1 where the product streams and 2 where
the gradient does), against the oracle at the operator's bars, with the kernels that ran; and the
choice of the image gradient made by timing what it runs."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import json, sys
import numpy as np, torch
sys.path.insert(0, sys.argv[1])
sys.path.insert(0, sys.argv[1] + "/tests")
from _common import Case, TOL, assert_close
T = lambda a: torch.from_numpy(np.ascontiguousarray(np.asarray(a).astype(np.complex64))).to("cuda:0")
H = lambda t: t.detach().cpu().numpy().astype(np.complex128)
ran = []
for kw in (dict(seed=511, dims=(48, 40), J=9, K=20, weights=True), dict(seed=512, dims=(30, 50), J=34, K=41),
           dict(seed=513, dims=(32, 36), J=6, K=13, mask="radial", spokes=9, weights=True)):
    cs = Case(**kw)
    for precision in ("fp32", "bf16_split"):
        print("[case]", kw, precision, flush=True)
        plan, tol = cs.plan(precision), TOL[precision]
        x, c, y = T(cs.x0), T(cs.c0), T(cs.y)
        maps = H(plan.basis_apply(c))
        B = np.asarray(cs.B)
        assert_close(maps, cs.c0 @ B.T, tol, coils=True, what="maps")
        assert_close(H(plan.basis_adjoint(T(maps))), maps.astype(np.complex64).astype(np.complex128) @ B.conj(), tol,
                     coils=True, what="basis adjoint")
        f, gx, gc = plan.grad(x, c, y)
        f_ref, gx_ref, gc_ref = cs.op.loss_and_grad(cs.x0, cs.c0, cs.y, cs.w)
        assert abs(float(f) - f_ref) <= tol * f_ref
        assert_close(H(gx).reshape(-1), gx_ref, tol, what="grad gx")
        assert_close(H(gc), gc_ref, tol, coils=True, what="grad gc")
        gx_ref, gc_ref = cs.op.adjoint(cs.x0, cs.c0, cs.y)
        plan.set_timing(True)
        gx, gc = plan.adjoint(x, c, y)
        torch.cuda.synchronize()
        ran.append(sorted(plan.timing()))
        plan.set_timing(False)
        assert_close(H(gx).reshape(-1), gx_ref, tol, what="gx")
        assert_close(H(gc), gc_ref, tol, coils=True, what="gc")
        gx, _ = plan.adjoint(x, c, y, want_gc=False)
        assert_close(H(gx).reshape(-1), gx_ref, tol, what="gx alone")
        _, gc = plan.adjoint(x, c, y, want_gx=False)
        assert_close(H(gc), gc_ref, tol, coils=True, what="gc alone")
print("RESULT " + json.dumps(ran), flush=True)
"""

CHOICE = r"""
import json, sys
import numpy as np, torch
sys.path.insert(0, sys.argv[1])
from paper_2008_09042_amd.encoding import MaxwellPlan
N, J, K = 64 * 64, 256, 300
g = lambda *s: torch.view_as_complex(torch.randn(*s, 2, device="cuda:0"))
plan = MaxwellPlan((64, 64), J, B=g(N, K), mask_idx=np.arange(0, N, 4))
plan.set_timing(True)
plan.adjoint(g(64, 64), g(J, K), g(J, plan.M))
torch.cuda.synchronize()
print("RESULT " + json.dumps(sorted(plan.timing())), flush=True)
"""


def run_child(code, cache):
    env = dict(os.environ, MAXWELL_TUNE_CACHE=cache)
    env.pop("MAXWELL_GEMM_AUTOTUNE", None)
    r = subprocess.run([sys.executable, "-c", code, ROOT], capture_output=True, text=True, env=env, timeout=110)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    line = [l for l in r.stdout.splitlines() if l.startswith("RESULT ")][-1]
    return json.loads(line[len("RESULT "):])


def test_each_choice_with_the_others_opposite(tmp_path):
    cache = str(tmp_path / "tune.txt")
    print("[case] choices by timing", flush=True)
    run_child(CHILD, cache)
    keys = [l.rsplit(" = ", 1)[0] for l in open(cache).read().splitlines()]
    assert len(keys) == 12
    # maps 1, image gradient 2; adjoint 1, coefficients' gradient 2
    for maps, adjoint in ((0, 0), (1, 2), (2, 1), (3, 0), (0, 3)):
        print(f"[case] choices {maps} {adjoint}", flush=True)
        with open(cache, "w") as f:
            for k in keys:
                v = maps if k.startswith("maps") else adjoint
                f.write(f"{k} = {4 * 2 + v}\n")
        for ran in run_child(CHILD, cache):
            assert ("dense_gx" in ran) == bool(maps & 2), ran
            # the combination runs for gx from maps, and for h where the adjoint does not form it
            assert ("adjoint_combine" in ran) == (not maps & 2 or not adjoint & 2), ran
            assert ("gemm_dense_apply" in ran) == (not maps & 2), ran


def test_image_gradient_chosen_by_what_it_runs(tmp_path):
    # few rows, many coils: maps and their combination take about two thirds of the streamed time
    print("[case] 64 x 64, 256 coils, 300 columns", flush=True)
    ran = run_child(CHOICE, str(tmp_path / "tune.txt"))
    assert "dense_gx" not in ran and "adjoint_combine" in ran, ran
