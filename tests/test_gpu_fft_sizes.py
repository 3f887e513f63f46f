"""Axis transforms at every radix of the two-radix kernel and at its limits, against the oracle.

The image sizes take each radix from 2 to 32 on the contiguous and on the strided axis, sizes
with one line per tile and tiles cut by the image, sizes that the pass-by-pass kernel keeps
(2 and above 1024), and the gridding window's passes at even and odd radices.  The bar is the
operator's: 1e-5 relative error (FP32 transforms of a few radix stages, about 1e-7 each).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from oracle.admm import sense_normal  # noqa: E402
from _common import assert_close  # noqa: E402

DEV = "cuda:0"


def c64(a):
    return np.asarray(a).astype(np.complex64).astype(np.complex128)


def run(dims, J, rng, **sampling):
    from paper_2008_09042_amd.encoding import MaxwellPlan
    N, K = int(np.prod(dims)), 3
    cg = lambda *s: c64(rng.normal(size=s) + 1j * rng.normal(size=s))  # noqa: E731
    B, x, c = cg(N, K), cg(*dims), cg(J, K)
    op = Oracle(dims, B=B, **sampling)
    plan = MaxwellPlan(dims, J, B=B, precision="fp32", device=DEV, **sampling)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a.astype(np.complex64))).to(DEV)  # noqa: E731
    H = lambda t: t.detach().cpu().numpy().astype(np.complex128)  # noqa: E731
    y = cg(J, plan.M)
    print(f"[case] {dims} J {J} M {plan.M}", flush=True)
    e = H(plan.encode(T(x), T(c)))
    gx, gc = plan.adjoint(T(x), T(c), T(y))
    gx_ref, gc_ref = op.adjoint(x, c, y)
    assert_close(e, op.encode(x, c), 1e-5, coils=True)
    assert_close(H(gx).reshape(-1), gx_ref, 1e-5)
    assert_close(H(gc), gc_ref, 1e-5, coils=True)
    S = cg(J, N)  # the masked round trip along the first axis, or the two transforms
    assert_close(H(plan.sense_normal(T(S), T(x))).reshape(-1), sense_normal(op, S, x), 1e-5)


CART = [(2, 4), (4, 2), (6, 16), (10, 18), (12, 20), (24, 30), (36, 64), (54, 50), (80, 90), (100, 108), (120, 144),
        (162, 6), (6, 162), (250, 4), (4, 250), (486, 2), (2, 486), (600, 4), (8, 512), (640, 8), (900, 2), (10, 1024),
        (1024, 6), (1200, 4), (4, 1200), (12, 10, 6), (18, 6, 32), (4, 320, 2)]


@pytest.mark.parametrize("dims", CART)
def test_cartesian(dims):
    rng = np.random.default_rng([31, *dims])
    N = int(np.prod(dims))
    mask = np.sort(rng.choice(N, size=max(1, N // 3), replace=False)).astype(np.int64)
    run(dims, 3, rng, mask_idx=mask)


@pytest.mark.parametrize("dims,sigma", [((16, 24), 2.0), ((24, 18), 2.0), ((90, 30), 2.0), ((20, 36), 1.5),
                                        ((40, 48), 1.25), ((600, 8), 2.0)])
def test_gridding_window(dims, sigma):
    rng = np.random.default_rng([32, *dims])
    traj = np.stack([rng.uniform(-n / 2, n / 2 * 0.999, size=257) for n in dims], axis=1)
    run(dims, 5, rng, traj=traj.astype(np.float32).astype(np.float64), oversamp=sigma)
