"""Dense basis products by the streaming kernels at the edges of their tiles, against NumPy.

Coil counts around the 16-coil blocks and past the 64-coil group, column counts that are odd
(8-byte rows), no multiple of 4 or 16, more than one workgroup's, and more fragments than LDS
holds at a time, images smaller than a workgroup's rows and cut by them.  The bars are the
operator's: 1e-5 in FP32, 1e-4 in BF16-split.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from _common import TOL, assert_close  # noqa: E402

DEV = "cuda:0"
SHAPES = [((2, 2), 1, 1), ((6, 10), 1, 3), ((16, 18), 7, 17), ((10, 6), 16, 16), ((24, 30), 17, 50), ((30, 36), 5, 75),
          ((32, 40), 33, 20), ((18, 16), 65, 12), ((20, 24), 100, 33), ((16, 50), 8, 130), ((12, 16), 20, 258),
          ((8, 12), 40, 600), ((256, 256), 3, 6), ((258 - 2, 270), 34, 9)]


@pytest.mark.parametrize("precision", ["fp32", "bf16_split"])
@pytest.mark.parametrize("dims,J,K", SHAPES)
def test_stream_products(dims, J, K, precision, monkeypatch):
    from paper_2008_09042_amd.encoding import MaxwellPlan
    monkeypatch.setenv("MAXWELL_GEMM_AUTOTUNE", "0")  # the streaming kernels, whatever is faster
    rng = np.random.default_rng([51, J, K, *dims])
    N = int(np.prod(dims))
    cg = lambda *s: (rng.normal(size=s) + 1j * rng.normal(size=s)).astype(np.complex64)  # noqa: E731
    B, c, h, x = cg(N, K), cg(J, K), cg(J, N), cg(*dims)
    mask = np.arange(N, dtype=np.int64)
    print(f"[case] {dims} J {J} K {K} {precision}", flush=True)
    plan = MaxwellPlan(dims, J, B=B, mask_idx=mask, precision=precision, device=DEV)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    H = lambda t: t.detach().cpu().numpy().astype(np.complex128)  # noqa: E731
    z = lambda a: a.astype(np.complex128)  # noqa: E731
    tol = TOL[precision]
    assert_close(H(plan.basis_apply(T(c))), z(c) @ z(B).T, tol, coils=True)
    assert_close(H(plan.basis_adjoint(T(h))), z(h) @ z(B).conj(), tol, coils=True)
    gx, gc = plan.adjoint(T(x), T(c), T(h))  # every point sampled: the samples are a k-space per coil
    gx_ref, gc_ref = Oracle(dims, B=z(B), mask_idx=mask).adjoint(z(x), z(c), z(h))
    assert_close(H(gx).reshape(-1), gx_ref, tol)
    assert_close(H(gc), gc_ref, tol, coils=True)
    # a misaligned basis and coil image: the 8-byte loads
    if N * K < 10000:
        Bt = torch.empty(N * K + 1, dtype=torch.complex64, device=DEV)[1:].view(N, K)
        Bt.copy_(T(B))
        ht = torch.empty(J * N + 1, dtype=torch.complex64, device=DEV)[1:].view(J, N)
        ht.copy_(T(h))
        odd = MaxwellPlan(dims, J, B=Bt, mask_idx=mask, precision=precision, device=DEV)
        assert odd.B.data_ptr() % 16 == 8
        assert_close(H(odd.basis_apply(T(c))), z(c) @ z(B).T, tol, coils=True)
        assert_close(H(odd.basis_adjoint(ht)), z(h) @ z(B).conj(), tol, coils=True)
