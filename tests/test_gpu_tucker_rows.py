"""General 3D Tucker path around the coil images, against the oracle: row and readout tiles cut
by the image, one to eight tiles of the readout, ranks of one to three tiles, one coil and many,
either gradient alone, maps and their adjoint at an 8-byte aligned stack, and the sizes just past
the limits (readout 130, rank 49), which keep the chain of products.  The bars are the
operator's: 1e-5 in FP32, 1e-4 in BF16-split."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from _common import TOL, assert_close  # noqa: E402

DEV = "cuda:0"
CASES = [((6, 4, 2), (2, 1, 1), 1), ((10, 16, 16), (3, 16, 16), 3), ((4, 18, 18), (4, 17, 5), 2),
         ((6, 30, 64), (2, 15, 33), 9), ((12, 32, 72), (5, 32, 20), 4), ((4, 100, 90), (3, 20, 16), 3),
         ((6, 48, 108), (2, 33, 48), 2), ((2, 50, 128), (2, 48, 17), 5), ((4, 54, 128), (3, 40, 40), 3),
         ((6, 20, 150), (2, 7, 9), 3), ((4, 54, 20), (3, 49, 6), 2), ((4, 10, 54), (2, 6, 49), 2)]


@pytest.mark.parametrize("precision", ["fp32", "bf16_split"])
@pytest.mark.parametrize("dims,ranks,J", CASES)
def test_tucker_rows(dims, ranks, J, precision):
    from paper_2008_09042_amd.encoding import MaxwellPlan
    rng = np.random.default_rng([71, J, *dims])
    cg = lambda *s: (rng.normal(size=s) + 1j * rng.normal(size=s)).astype(np.complex64)  # noqa: E731
    z = lambda a: np.asarray(a).astype(np.complex128)  # noqa: E731
    N, K = int(np.prod(dims)), 4
    U = [np.linalg.qr(z(cg(n, r)))[0].astype(np.complex64) for n, r in zip(dims, ranks)]
    core = (cg(*ranks, K) / np.sqrt(np.prod(ranks))).astype(np.complex64)
    x, c = cg(*dims), cg(J, K)
    mask = np.sort(rng.choice(N, size=max(3, N // 4), replace=False)).astype(np.int64)
    y, S = cg(J, mask.size), cg(J, N)
    op = Oracle(dims, U=[z(u) for u in U], core=z(core), mask_idx=mask)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    H = lambda t: t.detach().cpu().numpy().astype(np.complex128)  # noqa: E731
    tol = TOL[precision]
    print(f"[case] {dims} ranks {ranks} J {J} {precision}", flush=True)
    plan = MaxwellPlan(dims, J, U=U, core=core, mask_idx=mask, precision=precision, device=DEV)
    f_ref, gx_ref, gc_ref = op.loss_and_grad(z(x), z(c), z(y))
    f, gx, gc = plan.grad(T(x), T(c), T(y))
    assert abs(float(f) - f_ref) <= tol * f_ref
    assert_close(H(gx).reshape(-1), gx_ref, tol, what="gx")
    assert_close(H(gc), gc_ref, tol, coils=True, what="gc")
    gx_ref, gc_ref = op.adjoint(z(x), z(c), z(y))
    scale = torch.tensor(0.5, dtype=torch.float32, device=DEV)
    gx, _ = plan.adjoint(T(x), T(c), T(y), alpha=3.0, scale=scale, want_gc=False)
    assert_close(H(gx).reshape(-1), 1.5 * gx_ref, tol, what="gx alone")
    _, gc = plan.adjoint(T(x), T(c), T(y), alpha=3.0, scale=scale, want_gx=False)
    assert_close(H(gc), 1.5 * gc_ref, tol, coils=True, what="gc alone")
    assert_close(H(plan.encode(T(x), T(c))), op.encode(z(x), z(c)), tol, coils=True, what="encode")
    # a stack and an image that are aligned to one complex value
    off = lambda a: torch.cat([torch.zeros(1, dtype=torch.complex64, device=DEV), T(a).reshape(-1)])[1:].view(a.shape)  # noqa: E731
    ref = np.stack([op.basis_adjoint_one(s.reshape(dims)) for s in z(S)])
    assert_close(H(plan.basis_adjoint(T(S))), ref, tol, coils=True, what="basis adjoint")
    assert_close(H(plan.basis_adjoint(off(S))), ref, tol, coils=True, what="basis adjoint, 8-byte aligned")
    maps = np.stack([op.coil_map(cj).reshape(-1) for cj in z(c)])
    assert_close(H(plan.basis_apply(T(c))).reshape(J, N), maps, tol, coils=True, what="maps")
    gx, gc = plan.adjoint(off(x), T(c), off(y))
    assert_close(H(gx).reshape(-1), gx_ref, tol, what="gx, 8-byte aligned")
    assert_close(H(gc), gc_ref, tol, coils=True, what="gc, 8-byte aligned")
