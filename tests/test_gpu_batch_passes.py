"""A batch whose phases launch both forms of the transform for several slices at once: axes and grids
that do not split into two radices of at most 32 (972, 1000, 1200) beside some that do, Cartesian and
radial, on one branch.  Against the oracle at the operator's bars, and equal bit for bit to the
slices' own calls; also as replays of a captured graph."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from _common import TOL, Case, assert_close  # noqa: E402

DEV = "cuda:0"
SLICES = [dict(seed=601, dims=(972, 4), J=3, K=5, weights=True), dict(seed=602, dims=(4, 1200), J=2, K=6),
          dict(seed=603, dims=(500, 8), J=4, K=5, mask="radial", spokes=5, n_read=64, weights=True),
          dict(seed=604, dims=(8, 600), J=3, K=4, mask="radial", spokes=7, n_read=48),
          dict(seed=605, dims=(32, 48), J=4, K=7), dict(seed=606, dims=(1200, 6), J=5, K=4),
          dict(seed=607, dims=(64, 512), J=2, K=5, weights=True)]


@pytest.mark.parametrize("precision", ["fp32", "bf16_split"])
def test_both_transform_forms_in_one_phase(precision):
    from paper_2008_09042_amd.encoding import MaxwellBatch
    T = lambda a: torch.from_numpy(np.ascontiguousarray(np.asarray(a).astype(np.complex64))).to(DEV)  # noqa: E731
    H = lambda t: t.detach().cpu().numpy().astype(np.complex128)  # noqa: E731
    tol = TOL[precision]
    cases = [Case(**kw) for kw in SLICES]
    print(f"[case] {len(cases)} slices {precision}", flush=True)
    plans = [cs.plan(precision) for cs in cases]
    xs, cc, ys = ([T(getattr(cs, a)) for cs in cases] for a in ("x0", "c0", "y"))
    batch = MaxwellBatch(plans, branches=1)
    loss, gx, gc = batch.grad(xs, cc, ys)
    for i, (cs, plan) in enumerate(zip(cases, plans)):
        f_ref, gx_ref, gc_ref = cs.op.loss_and_grad(cs.x0, cs.c0, cs.y, cs.w)
        assert abs(float(loss[i]) - f_ref) <= tol * f_ref
        assert_close(H(gx[i]).reshape(-1), gx_ref, tol, what=f"gx {i}")
        assert_close(H(gc[i]), gc_ref, tol, coils=True, what=f"gc {i}")
        f1, gx1, gc1 = plan.grad(xs[i], cc[i], ys[i])
        assert torch.equal(f1, loss[i]) and torch.equal(gx1, gx[i]) and torch.equal(gc1, gc[i]), i
    want = (loss.clone(), [t.clone() for t in gx], [t.clone() for t in gc])
    batch.capture(xs, cc, ys)
    for _ in range(3):
        loss, gx, gc = batch.replay()
        torch.cuda.synchronize()
        assert torch.equal(loss, want[0])
        assert all(torch.equal(a, b) for a, b in zip(gx, want[1])) and all(torch.equal(a, b) for a, b in zip(gc, want[2]))
        plans[0].grad(xs[0], cc[0], ys[0])  # eager work between the replays
        for t in gx + gc:
            t.zero_()
