"""Gather and scatter-reduce bit for bit on either side of the lines that depend on
how rows lie in 64-byte granules and 128-byte lines: packed rows of 120 MB (78 MB
where they are not whole granules), and slab rows of 220 MB (128 MB of a larger
slab)."""
import pytest

from test_gpu_pack_hints import DEV, MB, _plan, _say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("limit,kz", [(120, 32), (120, 16), (120, 48), (78, 40)])
def test_packed_rows(limit, kz, over):
    n = limit * MB // (4 * kz) + over
    spc, plan = _plan(n)
    _say(f"packed lines: n={n} kz={kz}")
    S = torch.rand((2 * n, kz + 4), device=DEV,
                   generator=torch.Generator(device=DEV).manual_seed(n))
    assert torch.equal(spc.gather(plan, spc.ROWS, S, 4, kz), S[::2, 4:])


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("limit,kz,ld", [(128, 32, 64), (128, 32, 128), (128, 32, 80),
                                         (128, 16, 64), (220, 16, 64), (220, 64, 64)])
def test_slab_rows(limit, kz, ld, over):
    n = limit * MB // (4 * kz) + over
    spc, plan = _plan(n)
    _say(f"slab lines: n={n} kz={kz} ld={ld}")
    g = torch.Generator(device=DEV).manual_seed(n)
    packed = torch.rand((n, kz), device=DEV, generator=g)
    dst = torch.rand((2 * n, ld), device=DEV, generator=g)
    want = dst.clone()
    want[::2, ld - kz:] += packed
    spc.scatter_reduce(plan, spc.ROWS, packed, dst, ld - kz)
    assert torch.equal(dst, want)
