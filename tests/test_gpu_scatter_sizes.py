"""Scatter-reduce bit for bit on either side of the sizes from which it reads
(32 MB) and stores (128 MB) the slab past the caches: one FP32 addition an
element, so exact."""
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]

DEV = "cuda:0"


@pytest.mark.parametrize("kz", [32, 33])
@pytest.mark.parametrize("limit", [32 << 20, 128 << 20])
@pytest.mark.parametrize("over", [-1, 0, 1])
def test_around_the_streaming_sizes(kz, limit, over):
    from paper_2404_19638_amd import spc3d as spc
    n = limit // (4 * kz) + over
    ids = torch.arange(n, device=DEV) * 2   # every other row of the slab
    plan = spc.plan_create_coo(ids, torch.arange(n, device=DEV) % 97, (0, 2 * n), (0, 97))
    print(f"scatter: n={plan.R} kz={kz} bytes={4 * n * kz}", file=sys.stderr, flush=True)
    g = torch.Generator(device=DEV).manual_seed(n)
    packed = torch.rand((n, kz), device=DEV, generator=g)
    dst = torch.rand((2 * n, kz + 4), device=DEV, generator=g)
    want = dst.clone()
    want[::2, 4:] += packed
    for _ in range(2):
        got = spc.scatter_reduce(plan, spc.ROWS, packed, dst.clone(), 4)
        assert torch.equal(got, want)
