"""TV prox of 3D images whose workgroups are a quarter, half and all of the usual size (the image's
pixels decide), against the oracle (the prox's dual steps are nonexpansive: the operator's bar, 1e-5)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle.admm import tv_prox  # noqa: E402
from _common import rel  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("dims", [(18, 36, 10), (64, 30, 24), (60, 60, 18), (64, 64, 8), (8, 2, 16)])
def test_small_images(dims):
    from paper_2008_09042_amd.encoding import MaxwellPlan
    print(f"[case] {dims}", flush=True)
    rng = np.random.default_rng([61, *dims])
    N = int(np.prod(dims))
    z = (rng.normal(size=dims) + 1j * rng.normal(size=dims)).astype(np.complex64)
    B = torch.full((N, 1), 1.0 / np.sqrt(N), dtype=torch.complex64, device=DEV)
    plan = MaxwellPlan(dims, 1, B=B, mask_idx=np.arange(0, N, 7), precision="fp32", device=DEV)
    x = plan.tv_prox(torch.from_numpy(z).to(DEV), 0.3, 5).cpu().numpy().astype(np.complex128)
    ref = tv_prox(z.astype(np.complex128), float(np.float32(0.3)), 5)
    assert rel(x.reshape(-1), ref.reshape(-1)) <= 1e-5
