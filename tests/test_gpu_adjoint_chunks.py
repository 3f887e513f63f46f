"""The dense adjoint's split into column groups and row chunks: columns on both sides of one and
two groups per workgroup, images of a few rows and of several steps per chunk, against NumPy (the
bars are the operator's), and the row chunks' partials of a short basis below the basis itself."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from _common import TOL, assert_close  # noqa: E402

DEV = "cuda:0"


def problem(dims, J, K, precision, monkeypatch):
    from paper_2008_09042_amd.encoding import MaxwellPlan
    monkeypatch.setenv("MAXWELL_GEMM_AUTOTUNE", "0")  # the streaming kernels
    rng = np.random.default_rng([53, J, K, *dims])
    N = int(np.prod(dims))
    cg = lambda *s: (rng.normal(size=s) + 1j * rng.normal(size=s)).astype(np.complex64)  # noqa: E731
    B, h = cg(N, K), cg(J, N)
    print(f"[case] {dims} J {J} K {K} {precision}", flush=True)
    return MaxwellPlan(dims, J, B=B, mask_idx=np.arange(0, N, 3), precision=precision, device=DEV), B, h


@pytest.mark.parametrize("precision", ["fp32", "bf16_split"])
@pytest.mark.parametrize("dims,J,K", [((6, 6), 5, 64), ((6, 6), 5, 65), ((40, 36), 16, 128), ((40, 36), 16, 129),
                                      ((50, 60), 20, 192), ((24, 18), 20, 200), ((24, 18), 40, 32), ((40, 50), 40, 64),
                                      ((40, 50), 40, 65), ((64, 72), 70, 97), ((2, 2), 3, 300)])
def test_column_groups(dims, J, K, precision, monkeypatch):
    plan, B, h = problem(dims, J, K, precision, monkeypatch)
    c = plan.basis_adjoint(torch.from_numpy(h).to(DEV)).cpu().numpy().astype(np.complex128)
    assert_close(c, h.astype(np.complex128) @ B.astype(np.complex128).conj(), TOL[precision], coils=True)


def test_partials_of_a_short_basis_stay_below_the_basis(monkeypatch):
    plan, B, h = problem((64, 64), 17, 300, "fp32", monkeypatch)
    assert plan.ws_bytes < B.nbytes, plan.ws_bytes  # all of the workspace, the partials in it
