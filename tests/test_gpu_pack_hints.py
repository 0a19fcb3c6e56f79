"""Gather and scatter-reduce bit for bit on either side of the sizes from which
they read or store past the caches: source rows of 12 MB (32 MB where they are
converted), packed rows of 64 and 128 MB, slab rows of 32 and 256 MB, the last
on whole 64-byte granules only."""
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]

DEV = "cuda:0"
MB = 1 << 20


def _plan(n):
    from paper_2404_19638_amd import spc3d as spc
    ids = torch.arange(n, device=DEV) * 2   # every other row
    return spc, spc.plan_create_coo(ids, torch.arange(n, device=DEV) % 97, (0, 2 * n), (0, 97))


def _say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("limit,kz,src,packed", [
    (12, 32, torch.float32, torch.float32), (12, 30, torch.float32, torch.float32),
    (12, 64, torch.bfloat16, torch.bfloat16), (12, 64, torch.float32, torch.bfloat16),
    (32, 64, torch.float32, torch.bfloat16), (64, 30, torch.float32, torch.float32),
    (64, 32, torch.float32, torch.float32), (128, 64, torch.bfloat16, torch.bfloat16),
    (128, 36, torch.float32, torch.bfloat16)])
def test_gather_around_the_lines(limit, kz, src, packed, over):
    size = 2 if src == torch.bfloat16 else 4
    n = limit * MB // (size * kz) + over
    spc, plan = _plan(n)
    _say(f"gather hints: n={n} kz={kz} {src} to {packed}")
    g = torch.Generator(device=DEV).manual_seed(n)
    S = torch.rand((2 * n, kz + 2), device=DEV, generator=g).to(src)
    got = spc.gather(plan, spc.ROWS, S, 1, kz, packed)
    assert torch.equal(got, S[::2, 1:1 + kz].to(packed))


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("limit", [32, 256])
@pytest.mark.parametrize("kz,k0,ld,at", [(32, 16, 64, 0), (48, 0, 48, 0), (32, 16, 64, 4),
                                         (40, 0, 48, 0)])
def test_scatter_around_the_lines(limit, kz, k0, ld, at, over):
    n = limit * MB // (4 * kz) + over
    spc, plan = _plan(n)
    _say(f"scatter hints: n={n} kz={kz} k0={k0} ld={ld} at={at}")
    g = torch.Generator(device=DEV).manual_seed(n)
    packed = torch.rand((n, kz), device=DEV, generator=g)
    dst = torch.rand(2 * n * ld + at, device=DEV, generator=g)[at:].view(2 * n, ld)
    want = dst.clone()
    want[::2, k0:k0 + kz] += packed
    spc.scatter_reduce(plan, spc.ROWS, packed, dst, k0)
    assert torch.equal(dst, want)
