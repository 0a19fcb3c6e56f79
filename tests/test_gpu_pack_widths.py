"""Gather and scatter-reduce bit for bit against the oracle at every kind of
width: narrower than a 16-byte chunk, a multiple of one, between two (the last
chunk moved back over its neighbour), at odd column offsets and odd row
strides, with one row, a partial last wavefront, and enough rows for the
nontemporal stores."""
import sys

import numpy as np
import pytest

import oracle
from paper_2404_19638_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]

DEV = "cuda:0"


def _np(t):
    return t.detach().cpu().numpy()


def _check(n, used, kz, k0, K):
    from paper_2404_19638_amd import spc3d as spc
    rows = np.sort(np.random.default_rng(n + kz).choice(n, used, replace=False)).astype(np.int64)
    plan = spc.plan_create_coo(torch.from_numpy(rows).to(DEV), torch.zeros_like(
        torch.from_numpy(rows)).to(DEV), (0, n), (0, 1))
    print(f"pack: n={n} used={used} kz={kz} k0={k0} K={K}", file=sys.stderr, flush=True)
    src = synth.dense_f32(5, 0, n, K)
    S = torch.from_numpy(src).to(DEV)
    want = oracle.gather_f32(rows, 0, src, k0, kz)
    got = spc.gather(plan, spc.ROWS, S, k0, kz)
    np.testing.assert_array_equal(_np(got), want)
    got = spc.gather(plan, spc.ROWS, S, k0, kz, torch.bfloat16)
    np.testing.assert_array_equal(_np(got.view(torch.int16)).view(np.uint16),
                                  oracle.bf16_rne(want))
    H = S.bfloat16()
    got = spc.gather(plan, spc.ROWS, H, k0, kz, torch.bfloat16)
    assert torch.equal(got, H[torch.from_numpy(rows).to(DEV), k0:k0 + kz])
    packed = synth.dense_f32(6, 0, used, kz)
    slab = src.copy()
    oracle.scatter_add_f32(rows, 0, packed, slab, k0)
    spc.scatter_reduce(plan, spc.ROWS, torch.from_numpy(packed).to(DEV), S, k0)
    np.testing.assert_array_equal(_np(S).view(np.uint32), slab.view(np.uint32))


@pytest.mark.parametrize("kz", [1, 3, 4, 5, 7, 8, 9, 15, 16, 30, 33, 60, 127, 256, 1023, 1024])
@pytest.mark.parametrize("used", [1, 333])
def test_widths_and_offsets(kz, used):
    _check(1000, used, kz, 0, kz)
    _check(1000, used, kz, 3, kz + 4)


@pytest.mark.parametrize("used,kz", [(300_000, 32), (1_100_000, 32), (600_000, 61)])
def test_enough_rows_for_streamed_stores(used, kz):
    _check(1_300_000, used, kz, 1, kz + 2)
