"""Core contractions of small cores, whose reduction is split into parts of a chunk and whose
forward takes one row block per wave, against the oracle: one chunk and several, rows cut by the
last, each number of coil blocks, columns of one tile and more.  The bars are the operator's:
1e-5 in FP32, 1e-4 in BF16-split."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from _common import TOL, assert_close  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("precision", ["fp32", "bf16_split"])
@pytest.mark.parametrize("dims,ranks,J,K", [((6, 10, 12), (2, 2, 3), 1, 5), ((20, 18, 24), (8, 8, 8), 16, 40),
                                            ((20, 18, 24), (10, 9, 12), 17, 130), ((16, 32, 10), (11, 13, 5), 33, 33),
                                            ((36, 32, 30), (16, 16, 20), 50, 17), ((48, 48, 40), (24, 24, 20), 12, 120)])
def test_small_cores(dims, ranks, J, K, precision):
    from paper_2008_09042_amd.encoding import MaxwellPlan
    rng = np.random.default_rng([91, J, K, *dims])
    cg = lambda *s: (rng.normal(size=s) + 1j * rng.normal(size=s)).astype(np.complex64)  # noqa: E731
    z = lambda a: np.asarray(a).astype(np.complex128)  # noqa: E731
    U = [np.linalg.qr(z(cg(n, r)))[0].astype(np.complex64) for n, r in zip(dims, ranks)]
    core = (cg(*ranks, K) / np.sqrt(np.prod(ranks))).astype(np.complex64)
    npl = dims[0] * dims[1]
    lines = np.sort(rng.choice(npl, size=npl // 5, replace=False))
    mask = (lines[:, None] * dims[2] + np.arange(dims[2])[None, :]).reshape(-1).astype(np.int64)
    x, c, y = cg(*dims), cg(J, K), cg(J, mask.size)
    op = Oracle(dims, U=[z(u) for u in U], core=z(core), mask_idx=mask)
    plan = MaxwellPlan(dims, J, U=U, core=core, mask_idx=mask, precision=precision, device=DEV)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    H = lambda t: t.detach().cpu().numpy().astype(np.complex128)  # noqa: E731
    print(f"[case] {dims} ranks {ranks} J {J} K {K} {precision} {plan.path}", flush=True)
    assert_close(H(plan.encode(T(x), T(c))), op.encode(z(x), z(c)), TOL[precision], coils=True, what="encode")
    gx_ref, gc_ref = op.adjoint(z(x), z(c), z(y))
    gx, gc = plan.adjoint(T(x), T(c), T(y))
    assert_close(H(gx).reshape(-1), gx_ref, TOL[precision], what="gx")
    assert_close(H(gc), gc_ref, TOL[precision], coils=True, what="gc")
