"""Maps of few columns over many rows (four blocks of 32 for every wave of 512 workgroups: 524288
rows): the last size of the general streaming kernel and the first of the one that goes through row
blocks, rows cut by a block, one and two blocks of coils, odd columns and a misaligned basis,
against float64 on the device.  The bars are the operator's."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from _common import TOL  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("precision", ["fp32", "bf16_split"])
@pytest.mark.parametrize("dims,J,K", [((750, 640), 2, 4), ((512, 1024), 1, 1), ((720, 750), 3, 5), ((720, 750), 16, 16),
                                      ((720, 750), 17, 15), ((1024, 1000), 32, 8), ((720, 750), 33, 8),
                                      ((720, 750), 4, 17)])
def test_narrow_maps(dims, J, K, precision, monkeypatch):
    from paper_2008_09042_amd.encoding import MaxwellPlan
    monkeypatch.setenv("MAXWELL_GEMM_AUTOTUNE", "0")  # the streaming kernels
    g = torch.Generator(device=DEV).manual_seed(J * 100 + K)
    N = dims[0] * dims[1]
    print(f"[case] {dims} J {J} K {K} {precision}", flush=True)
    flat = torch.view_as_complex(torch.randn(N * K + 1, 2, generator=g, device=DEV))
    c = torch.view_as_complex(torch.randn(J, K, 2, generator=g, device=DEV))
    for off in (0, 1):
        B = flat[off:off + N * K].view(N, K)  # with the offset, 8-byte aligned
        plan = MaxwellPlan(dims, J, B=B, mask_idx=[0, N - 1], precision=precision, device=DEV)
        assert plan.B.data_ptr() % 16 == 8 * off
        S = plan.basis_apply(c).to(torch.complex128)
        # columns summed one at a time: no batched product
        ref = sum(c[:, k:k + 1].to(torch.complex128) * B[:, k].to(torch.complex128)[None] for k in range(K))
        err, mag = (S - ref).abs(), ref.abs()
        assert float((err.square().sum() / mag.square().sum()).sqrt()) <= TOL[precision]
        assert float((err.amax(1) / mag.amax(1)).max()) <= TOL[precision]
