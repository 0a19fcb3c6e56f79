"""The one-pass attention forward on a block of more than 2^24 rows and
columns, where row offsets take 64 bits: with one entry per row each output
row is its value row exactly, whatever the score."""
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]

DEV = "cuda:0"


@pytest.mark.parametrize("dtype,kz", [(torch.bfloat16, 32), (torch.float32, 16)])
def test_more_rows_than_24_bits(dtype, kz):
    from paper_2404_19638_amd import spc3d as spc
    n = (1 << 24) + 77
    print(f"attention: n={n} kz={kz} {dtype}", file=sys.stderr, flush=True)
    rows = torch.arange(n, device=DEV)
    plan = spc.plan_create_coo(rows, n - 1 - rows, (0, n), (0, n))
    g = torch.Generator(device=DEV).manual_seed(3)
    Q, K, V = (torch.empty((n, kz), device=DEV).uniform_(-1, 1, generator=g).to(dtype)
               for _ in range(3))
    out, stats = spc.attention_fwd(plan, Q, K, V)
    assert torch.equal(out, V.float().flip(0))
    assert torch.equal(stats[:, 1], torch.ones(n, device=DEV))
