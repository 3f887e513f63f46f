"""The dense adjoint where three or four column groups over many rows take one workgroup: both
sides of the line, coil blocks of one, two and four, even and odd columns, and rows that end in a cut
step, alone and with conj(x) formed on the way, against NumPy (the bars are the operator's)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from _common import TOL, assert_close  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("precision", ["fp32", "bf16_split"])
@pytest.mark.parametrize("dims,J,K", [((512, 256), 3, 130), ((400, 324), 3, 130), ((486, 270), 17, 255), ((600, 250), 33, 65),
                                      ((486, 270), 4, 257)])
def test_many_rows(dims, J, K, precision, monkeypatch):
    from paper_2008_09042_amd.encoding import MaxwellPlan
    monkeypatch.setenv("MAXWELL_GEMM_AUTOTUNE", "0")  # the streaming kernels
    rng = np.random.default_rng([59, J, K, *dims])
    N = int(np.prod(dims))
    cg = lambda *s: (rng.standard_normal(s, np.float32) + 1j * rng.standard_normal(s, np.float32)).astype(np.complex64)  # noqa: E731
    B, h, x = cg(N, K), cg(J, N), cg(*dims)
    print(f"[case] {dims} J {J} K {K} {precision}", flush=True)
    plan = MaxwellPlan(dims, J, B=B, mask_idx=np.arange(N), precision=precision, device=DEV)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    H = lambda t: t.cpu().numpy().astype(np.complex128)  # noqa: E731
    Bc = B.astype(np.complex128).conj()
    assert_close(H(plan.basis_adjoint(T(h))), h.astype(np.complex128) @ Bc, TOL[precision], coils=True, what="basis adjoint")
    # the samples are the whole k-space: F_s^H is the inverse of F
    image = h.reshape(J, *dims).astype(np.complex128)
    y = np.fft.fftshift(np.fft.fft2(np.fft.ifftshift(image, axes=(1, 2)), norm="ortho"), axes=(1, 2)).reshape(J, N)
    _, gc = plan.adjoint(T(x), T(cg(J, K)), T(y.astype(np.complex64)), want_gx=False)
    ref = (np.conj(x.astype(np.complex128)).reshape(1, N) * h) @ Bc
    assert_close(H(gc), ref, TOL[precision], coils=True, what="gc")
