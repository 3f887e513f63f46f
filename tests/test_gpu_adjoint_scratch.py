"""Where the dense adjoint's partials live: in the maps' region, in the samples' and GEMMs', in a
region of their own, and as many row chunks as fit where that region would take the plan past
what maxwell_grad_static holds; against the oracle, at the operator's bars."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from _common import TOL, assert_close  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("precision", ["fp32", "bf16_split"])
@pytest.mark.parametrize("dims,J,K,static", [((32, 30), 3, 4, True), ((64, 64), 8, 150, True), ((96, 60), 20, 300, True),
                                             ((128, 128), 64, 500, True), ((100, 96), 128, 300, False)])
def test_adjoint_scratch(dims, J, K, static, precision, monkeypatch):
    from paper_2008_09042_amd.encoding import MaxwellPlan
    monkeypatch.setenv("MAXWELL_GEMM_AUTOTUNE", "0")  # the streaming kernels, whatever is faster
    rng = np.random.default_rng([101, J, K, *dims])
    N = int(np.prod(dims))
    cg = lambda *s: (rng.normal(size=s) + 1j * rng.normal(size=s)).astype(np.complex64)  # noqa: E731
    z = lambda a: np.asarray(a).astype(np.complex128)  # noqa: E731
    mask = np.sort(rng.choice(N, size=N // 5, replace=False)).astype(np.int64)
    B, x, c, y, h = cg(N, K), cg(*dims), cg(J, K), cg(J, mask.size), cg(J, N)
    plan = MaxwellPlan(dims, J, B=B, mask_idx=mask, precision=precision, device=DEV)
    print(f"[case] {dims} J {J} K {K} {precision} workspace {plan.ws_bytes}", flush=True)
    assert (plan.ws_bytes <= 64 << 20) == static
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    H = lambda t: t.detach().cpu().numpy().astype(np.complex128)  # noqa: E731
    tol = TOL[precision]
    f_ref, gx_ref, gc_ref = Oracle(dims, B=z(B), mask_idx=mask).loss_and_grad(z(x), z(c), z(y))
    f, gx, gc = plan.grad(T(x), T(c), T(y))
    assert abs(float(f) - f_ref) <= tol * f_ref
    assert_close(H(gx).reshape(-1), gx_ref, tol, what="gx")
    assert_close(H(gc), gc_ref, tol, coils=True, what="gc")
    assert_close(H(plan.basis_adjoint(T(h))), z(h) @ z(B).conj(), tol, coils=True, what="basis adjoint")
    gx, gc = plan.adjoint(T(x), T(c), T(y))
    r_gx, r_gc = Oracle(dims, B=z(B), mask_idx=mask).adjoint(z(x), z(c), z(y))
    assert_close(H(gx).reshape(-1), r_gx, tol, what="adjoint gx")
    assert_close(H(gc), r_gc, tol, coils=True, what="adjoint gc")
