"""Cartesian residual and loss formed inside the axis transforms, against the oracle.

The forward's last pass (residual written as samples) and the round trip of the gradient
(residual kept in registers) at even and odd radices, both size classes, tiles cut by the
image, one sampled point and all of them, with and without weights; 972 rows and the 1D image
keep the separate residual.  Bars: 1e-5 relative on arrays (FP32 transforms), and on the loss,
whose terms carry twice the relative error of their residuals.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from _common import assert_close  # noqa: E402

DEV = "cuda:0"
DIMS = [(2, 4), (6, 10), (30, 16), (50, 12), (36, 6), (54, 36), (64, 20), (90, 150), (250, 4), (288, 4), (432, 2), (486, 6),
        (750, 4), (1024, 6), (972, 4), (12, 10, 6), (20, 2, 18)]


def c64(a):
    return np.asarray(a).astype(np.complex64).astype(np.complex128)


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("dims", DIMS)
def test_residual_pass(dims, weighted):
    from paper_2008_09042_amd.encoding import MaxwellPlan
    rng = np.random.default_rng([41, weighted, *dims])
    N, K, J = int(np.prod(dims)), 3, 5
    M = {(2, 4): 1, (64, 20): N}.get(dims, max(2, N // 3))
    mask = np.sort(rng.permutation(N)[:M]).astype(np.int64)
    cg = lambda *s: c64(rng.normal(size=s) + 1j * rng.normal(size=s))  # noqa: E731
    B, x, c, y = cg(N, K), cg(*dims), cg(J, K), cg(J, M)
    w = rng.uniform(0.25, 2.0, size=M).astype(np.float32).astype(np.float64) if weighted else None
    op = Oracle(dims, B=B, mask_idx=mask)
    plan = MaxwellPlan(dims, J, B=B, mask_idx=mask, weights=w, precision="fp32", device=DEV)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a.astype(np.complex64))).to(DEV)  # noqa: E731
    H = lambda t: t.detach().cpu().numpy().astype(np.complex128)  # noqa: E731
    print(f"[case] {dims} M {M} weighted {weighted}", flush=True)
    f_ref, gx_ref, gc_ref = op.loss_and_grad(x, c, y, w)
    r_ref = (op.encode(x, c) - y) * (1.0 if w is None else w)
    args = T(x), T(c), T(y)
    r, loss = plan.forward_loss(*args)
    assert_close(H(r), r_ref, 1e-5, coils=True, what="r")
    assert abs(float(loss) / f_ref - 1) <= 2e-5
    _, loss = plan.forward_loss(*args, want_r=False)
    assert abs(float(loss) / f_ref - 1) <= 2e-5
    loss, gx, gc = plan.grad(*args)
    assert abs(float(loss) / f_ref - 1) <= 2e-5
    assert_close(H(gx).reshape(-1), np.asarray(gx_ref).reshape(-1), 1e-5, what="gx")
    assert_close(H(gc), gc_ref, 1e-5, coils=True, what="gc")
