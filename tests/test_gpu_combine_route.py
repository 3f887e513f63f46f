"""Where the SENSE normal operator sums over the coils in its last inverse pass: from 128 to 512 rows
(960 up to eight coils) of a last axis of two radices up to 16; with fewer or more the combination stays a
pass of its own.
Sizes on both sides of the lines, against the oracle at the operator's bar, 1e-5."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from oracle.admm import sense_normal  # noqa: E402
from _common import assert_close  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("dims,J,summed", [((120, 30), 3, False), ((128, 30), 3, True), ((512, 12), 5, True),
                                           ((512, 12), 9, True), ((540, 12), 9, False), ((540, 12), 8, True),
                                           ((960, 30), 5, True), ((1024, 16), 5, False), ((24, 24, 4), 9, False),
                                           ((24, 24, 4), 2, True), ((16, 32, 4), 2, True), ((30, 20, 256), 9, False),
                                           ((30, 20, 64), 2, True), ((16, 20, 128), 9, True), ((128, 288), 2, False)])
def test_combine_route(dims, J, summed):
    from paper_2008_09042_amd.encoding import MaxwellPlan
    rng = np.random.default_rng([112, J, *dims])
    N = int(np.prod(dims))
    cg = lambda *s: (rng.normal(size=s) + 1j * rng.normal(size=s)).astype(np.complex64)  # noqa: E731
    z = lambda a: np.asarray(a).astype(np.complex128)  # noqa: E731
    mask = np.sort(rng.choice(N, size=N // 3, replace=False)).astype(np.int64)
    B, S, x = cg(N, 2), cg(J, N), cg(*dims)
    plan = MaxwellPlan(dims, J, B=B, mask_idx=mask, precision="fp32", device=DEV)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    print(f"[case] {dims} J {J}", flush=True)
    plan.set_timing(True)
    out = plan.sense_normal(T(S), T(x))
    torch.cuda.synchronize()
    names = plan.timing()
    plan.set_timing(False)
    assert ("fft_combine" in names) == summed and ("adjoint_combine" in names) != summed, sorted(names)
    ref = sense_normal(Oracle(dims, B=z(B), mask_idx=mask), z(S), z(x))
    assert_close(out.cpu().numpy().astype(np.complex128).reshape(-1), np.asarray(ref).reshape(-1), 1e-5)
