"""Which way the general 3D Tucker path takes to the image gradient, and that both are right: maps
kept in registers where the image's rows fill the chip or the coils are few, maps in memory and
their combination elsewhere.  Sizes on both sides of the lines (512 blocks of 16 rows; four coils
in BF16-split, two in FP32), against the oracle; the bars are the operator's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from _common import TOL, assert_close  # noqa: E402

DEV = "cuda:0"
# dims, ranks, coils, whether the rows fill the chip (there also readouts and ranks of several tiles)
CASES = [((32, 250, 4), (3, 7, 4), 6, True), ((32, 240, 4), (3, 7, 4), 6, False), ((20, 20, 20), (3, 7, 4), 2, False),
         ((20, 20, 20), (3, 7, 4), 3, False), ((20, 20, 20), (3, 7, 4), 4, False), ((20, 20, 20), (3, 7, 4), 5, False),
         ((24, 24, 24), (5, 8, 20), 64, False), ((4, 30, 100), (3, 17, 40), 9, False),
         ((64, 120, 36), (2, 33, 16), 3, True), ((64, 120, 90), (2, 20, 18), 3, True),
         ((64, 120, 128), (2, 17, 40), 3, True)]


@pytest.mark.parametrize("precision", ["fp32", "bf16_split"])
@pytest.mark.parametrize("dims,ranks,J,rows_fill", CASES)
def test_gx_route(dims, ranks, J, rows_fill, precision):
    from paper_2008_09042_amd.encoding import MaxwellPlan
    rng = np.random.default_rng([72, J, *dims])
    cg = lambda *s: (rng.normal(size=s) + 1j * rng.normal(size=s)).astype(np.complex64)  # noqa: E731
    z = lambda a: np.asarray(a).astype(np.complex128)  # noqa: E731
    N, K = int(np.prod(dims)), 4
    U = [np.linalg.qr(z(cg(n, r)))[0].astype(np.complex64) for n, r in zip(dims, ranks)]
    core = (cg(*ranks, K) / np.sqrt(np.prod(ranks))).astype(np.complex64)
    x, c = cg(*dims), cg(J, K)
    mask = np.sort(rng.choice(N, size=N // 4, replace=False)).astype(np.int64)
    y = cg(J, mask.size)
    op = Oracle(dims, U=[z(u) for u in U], core=z(core), mask_idx=mask)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    H = lambda t: t.detach().cpu().numpy().astype(np.complex128)  # noqa: E731
    tol = TOL[precision]
    print(f"[case] {dims} J {J} {precision}", flush=True)
    plan = MaxwellPlan(dims, J, U=U, core=core, mask_idx=mask, precision=precision, device=DEV)
    assert plan.path != "fused-tucker-lines"
    registers = rows_fill or J <= (4 if precision == "bf16_split" else 2)
    plan.set_timing(True)
    f, gx, gc = plan.grad(T(x), T(c), T(y))
    torch.cuda.synchronize()
    assert ("adjoint_combine" not in plan.timing()) == registers, sorted(plan.timing())
    plan.set_timing(False)
    f_ref, gx_ref, gc_ref = op.loss_and_grad(z(x), z(c), z(y))
    assert abs(float(f) - f_ref) <= tol * f_ref
    assert_close(H(gx).reshape(-1), gx_ref, tol, what="gx")
    assert_close(H(gc), gc_ref, tol, coils=True, what="gc")
    gx_ref, gc_ref = op.adjoint(z(x), z(c), z(y))
    scale = torch.tensor(0.5, dtype=torch.float32, device=DEV)
    gx, gc = plan.adjoint(T(x), T(c), T(y), alpha=3.0, scale=scale)
    assert_close(H(gx).reshape(-1), 1.5 * gx_ref, tol, what="adjoint gx")
    assert_close(H(gc), 1.5 * gc_ref, tol, coils=True, what="adjoint gc")
    gx, _ = plan.adjoint(T(x), T(c), T(y), want_gc=False)
    assert_close(H(gx).reshape(-1), gx_ref, tol, what="gx alone")
    _, gc = plan.adjoint(T(x), T(c), T(y), want_gx=False)
    assert_close(H(gc), gc_ref, tol, coils=True, what="gc alone")
