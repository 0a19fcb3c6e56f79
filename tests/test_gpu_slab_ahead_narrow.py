"""FP32 rows of 9 to 16 values (4 lanes) on either side of the 10 entries a row below
which the folded pass reads destinations with a step's rows, ragged ones among them:
the slab ends bit for bit as the plain pass's rows added to it."""
import numpy as np
import pytest

import oracle
from paper_2404_19638_amd import synth
from test_gpu_run_family import DEV, Block, _np, _say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]


@pytest.mark.parametrize("kz", [9, 12, 13, 15, 16])
@pytest.mark.parametrize("nnz", [1, 9, 10 * 700 - 1, 10 * 700, 701])
def test_around_ten_entries_a_row(kz, nnz):
    rng = np.random.default_rng(nnz)
    n = min(700, nnz)
    rows = np.sort(np.concatenate([np.arange(n), rng.integers(0, n, nnz - n)]))
    cols = np.arange(nnz, dtype=np.int64) * 37 % 8009
    b = Block(rows, cols, n, 8009)
    spc, plan = b.spc, b.plan
    assert plan.R == n and plan.nnz == nnz
    _say(f"slab ahead, narrow: R={n} nnz={nnz} kz={kz}")
    b.check(kz, False, what="narrow")
    _, _, Ad, Bd = b.operands(kz, False, 62)
    out, Y = spc.sddmm_spmm(plan, b.v, Ad, Bd, kz)
    slab0 = synth.dense_f32(9, 0, n, kz)
    want = slab0.copy()
    oracle.scatter_add_f32(b.ref["gmap_r"], 0, _np(Y), want, 0)
    slab = torch.from_numpy(slab0).to(DEV)
    out2 = spc.sddmm_spmm_scatter(plan, b.v, Ad, Bd, slab, 0, kz)
    np.testing.assert_array_equal(_np(slab).view(np.uint32), want.view(np.uint32))
    assert torch.equal(out2, out)
