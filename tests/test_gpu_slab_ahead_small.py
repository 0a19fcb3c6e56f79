"""FP32 rows on 8 lanes on either side of the numbers of wavefronts (4096, 2048 with two
vectors a lane) and of entries a row (20) up to which the folded pass reads
destinations with a step's rows, ragged ones among them: the slab ends bit for bit
as the plain pass's rows added to it."""
import numpy as np
import pytest

import oracle
from paper_2404_19638_amd import synth
from test_gpu_run_family import DEV, Block, _np, _say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]


def _check(n, nnz, kz):
    rows = np.arange(nnz, dtype=np.int64) % n
    cols = (np.arange(nnz, dtype=np.int64) // n * 331 + rows * 7) % 9973
    b = Block(rows, cols, n, 9973)
    spc, plan = b.spc, b.plan
    assert plan.R == n and plan.nnz == nnz
    _say(f"slab ahead, small: R={n} nnz={nnz} kz={kz}")
    _, _, Ad, Bd = b.operands(kz, False, 62)
    out, Y = spc.sddmm_spmm(plan, b.v, Ad, Bd, kz)
    slab0 = synth.dense_f32(9, 0, n, kz + 3)
    want = slab0.copy()
    oracle.scatter_add_f32(b.ref["gmap_r"], 0, _np(Y), want, 2)
    slab = torch.from_numpy(slab0).to(DEV)
    out2 = spc.sddmm_spmm_scatter(plan, b.v, Ad, Bd, slab, 2, kz)
    np.testing.assert_array_equal(_np(slab).view(np.uint32), want.view(np.uint32))
    assert torch.equal(out2, out)


@pytest.mark.parametrize("kz", [17, 30, 32, 33, 40, 63, 64])
@pytest.mark.parametrize("n,nnz", [(1, 1), (7, 9), (301, 20 * 301 - 1), (301, 20 * 301)])
def test_few_entries(n, nnz, kz):
    _check(n, nnz, kz)


@pytest.mark.parametrize("kz,nnz", [(32, 4096 * 128), (30, 4096 * 128), (64, 2048 * 128),
                                    (63, 2048 * 128)])
@pytest.mark.parametrize("over", [-1, 0])
def test_around_the_wavefronts(kz, nnz, over):
    _check(40000, nnz + over, kz)
