"""SENSE normal operator with the coil sum in the last inverse pass, against the oracle: even and
odd radices, coil tiles cut by the last and filled by few coils, several transforms per line of
threads, 3D rows, and the sizes that keep the separate combination (few rows, a radix above 16).
The bar is the operator's, 1e-5."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from oracle.admm import sense_normal  # noqa: E402
from _common import assert_close  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("dims,J", [((128, 4), 1), ((128, 6), 3), ((144, 10), 70), ((150, 30), 5), ((128, 54), 17),
                                    ((160, 90), 33), ((256, 128), 9), ((128, 216), 4), ((128, 256), 32),
                                    ((12, 16, 20), 6), ((120, 64), 4), ((128, 320), 2)])
def test_combine_pass(dims, J):
    from paper_2008_09042_amd.encoding import MaxwellPlan
    rng = np.random.default_rng([111, J, *dims])
    N = int(np.prod(dims))
    cg = lambda *s: (rng.normal(size=s) + 1j * rng.normal(size=s)).astype(np.complex64)  # noqa: E731
    z = lambda a: np.asarray(a).astype(np.complex128)  # noqa: E731
    mask = np.sort(rng.choice(N, size=N // 3, replace=False)).astype(np.int64)
    B, S, x = cg(N, 2), cg(J, N), cg(*dims)
    plan = MaxwellPlan(dims, J, B=B, mask_idx=mask, precision="fp32", device=DEV)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    print(f"[case] {dims} J {J}", flush=True)
    out = plan.sense_normal(T(S), T(x)).detach().cpu().numpy().astype(np.complex128).reshape(-1)
    assert_close(out, np.asarray(sense_normal(Oracle(dims, B=z(B), mask_idx=mask), z(S), z(x))).reshape(-1), 1e-5)
