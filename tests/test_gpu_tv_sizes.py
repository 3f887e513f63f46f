"""TV prox on images at the edges of its tiles (16 x 16 pixels, five steps per launch), against
the oracle.  The prox's dual steps are nonexpansive, so FP32 rounding does not grow with the
step count: the bar is the operator's 1e-5."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle.admm import tv_prox  # noqa: E402
from _common import rel  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("dims", [(2, 2), (2, 30), (16, 16), (18, 32), (30, 50), (48, 2), (6, 10, 12)])
def test_tv_prox_tiles(dims):
    from paper_2008_09042_amd.encoding import MaxwellPlan
    rng = np.random.default_rng([41, *dims])
    N = int(np.prod(dims))
    z = (rng.normal(size=dims) + 1j * rng.normal(size=dims)).astype(np.complex64)
    B = np.full((N, 1), 1.0 / np.sqrt(N), dtype=np.complex64)
    plan = MaxwellPlan(dims, 1, B=B, mask_idx=np.arange(N, dtype=np.int64), precision="fp32", device=DEV)
    zt = torch.from_numpy(z).to(DEV)
    for iters in (0, 1, 4, 5, 6, 11):
        print(f"[case] {dims} {iters} steps", flush=True)
        x = plan.tv_prox(zt, 0.3, iters).cpu().numpy().astype(np.complex128)
        ref = tv_prox(z.astype(np.complex128), float(np.float32(0.3)), iters)
        assert rel(x.reshape(-1), ref.reshape(-1)) <= 1e-5, iters
