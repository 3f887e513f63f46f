"""Fused 3D path at every plane axis size and at readouts of one, two and three radices, against
the oracle: the gradient, the encoding and its adjoint, the Jacobian-vector product and the
normal operator with and without weights.  The bars are the operator's: 1e-5 in FP32, 1e-4 in
BF16-split."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from oracle.solver import normal  # noqa: E402
from _common import TOL, assert_close  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("precision", ["fp32", "bf16_split"])
@pytest.mark.parametrize("dims,ranks,J", [((16, 128, 10), (4, 9, 3), 5), ((128, 16, 6), (17, 5, 3), 2),
                                          ((96, 48, 18), (33, 20, 6), 3), ((48, 96, 100), (20, 40, 9), 4),
                                          ((80, 64, 250), (11, 8, 7), 2), ((64, 80, 162), (16, 16, 5), 3),
                                          ((32, 32, 2), (5, 4, 2), 7), ((64, 64, 48), (40, 33, 8), 2),
                                          ((128, 128, 4), (40, 36, 3), 3)])
def test_plane_and_readout_sizes(dims, ranks, J, precision):
    from paper_2008_09042_amd.encoding import MaxwellPlan
    rng = np.random.default_rng([61, J, *dims])
    cg = lambda *s: (rng.normal(size=s) + 1j * rng.normal(size=s)).astype(np.complex64)  # noqa: E731
    z = lambda a: np.asarray(a).astype(np.complex128)  # noqa: E731
    K = 4
    U = [np.linalg.qr(z(cg(n, r)))[0].astype(np.complex64) for n, r in zip(dims, ranks)]
    core = (cg(*ranks, K) / np.sqrt(np.prod(ranks))).astype(np.complex64)
    x, c, dx, dc = cg(*dims), cg(J, K), cg(*dims), cg(J, K)
    npl = dims[0] * dims[1]
    lines = np.sort(rng.choice(npl, size=max(3, npl // 5), replace=False))
    mask = (lines[:, None] * dims[2] + np.arange(dims[2])[None, :]).reshape(-1).astype(np.int64)
    w = rng.uniform(0.1, 1.0, size=mask.size).astype(np.float32)
    y = cg(J, mask.size)
    op = Oracle(dims, U=[z(u) for u in U], core=z(core), mask_idx=mask)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    H = lambda t: t.detach().cpu().numpy().astype(np.complex128)  # noqa: E731
    tol = TOL[precision]
    print(f"[case] {dims} ranks {ranks} J {J} {precision}", flush=True)
    for weights in (None, w):
        plan = MaxwellPlan(dims, J, U=U, core=core, mask_idx=mask, weights=weights, precision=precision, device=DEV)
        assert plan.path == "fused-tucker-lines"
        f, gx, gc = plan.grad(T(x), T(c), T(y))
        f_ref, gx_ref, gc_ref = op.loss_and_grad(z(x), z(c), z(y), weights)
        assert abs(float(f.item()) - f_ref) <= tol * f_ref
        assert_close(H(gx).reshape(-1), gx_ref, tol)
        assert_close(H(gc), gc_ref, tol, coils=True)
        lx, lc = 0.3, 0.7
        ox, oc = plan.normal(T(x), T(c), T(dx), T(dc), lx, lc)
        ox_ref, oc_ref = normal(op, z(x), z(c), z(dx), z(dc), float(np.float32(lx)), float(np.float32(lc)),
                                None if weights is None else weights.astype(np.float64))
        assert_close(H(ox).reshape(-1), np.asarray(ox_ref).reshape(-1), tol)
        assert_close(H(oc), oc_ref, tol, coils=True)
    assert_close(H(plan.jvp(T(x), T(c), T(dx), T(dc))), op.jvp(z(x), z(c), z(dx), z(dc)), tol, coils=True)
    gx, gc = plan.adjoint(T(x), T(c), T(y))
    gx_ref, gc_ref = op.adjoint(z(x), z(c), z(y))
    assert_close(H(gx).reshape(-1), gx_ref, tol)
    assert_close(H(gc), gc_ref, tol, coils=True)
