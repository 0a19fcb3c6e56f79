"""SpMM and the fused pass at ragged widths on either side of the 100 MB of Y from
which finished rows are stored past the caches, on rows of one entry: every Y
row is value times B row, bit for bit."""
import pytest

from test_gpu_run_family import DEV, _say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]


@pytest.mark.parametrize("kz,dtype", [(30, torch.float32), (50, torch.float32),
                                      (30, torch.bfloat16), (100, torch.bfloat16)])
@pytest.mark.parametrize("over", [0, 1])
def test_around_the_line(kz, dtype, over):
    from paper_2404_19638_amd import spc3d as spc
    n = (100 << 20) // (4 * kz) + over
    g = torch.Generator(device=DEV).manual_seed(n)
    rows = torch.arange(n, device=DEV)
    cols = rows * 7919 % 5003
    plan = spc.plan_create_coo(rows, cols, (0, n), (0, 5003))
    _say(f"ragged stores: R={plan.R} kz={kz} {dtype}")
    A = torch.rand((n, kz), device=DEV, generator=g).to(dtype)
    B = torch.rand((plan.C, kz), device=DEV, generator=g).to(dtype)
    v = torch.rand(n, device=DEV, generator=g)
    want = v[:, None] * B[plan.maps()["colidx"].long()].float()
    Y = torch.full((n, kz), float("nan"), device=DEV)
    assert torch.equal(spc.spmm(plan, v, B, 0, kz, out=Y), want)
    Y.fill_(float("nan"))
    _, Yf = spc.sddmm_spmm(plan, v, A, B, kz, Y=Y)
    assert torch.equal(Yf, want)
