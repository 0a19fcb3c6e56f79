"""SpMM and the fused pass with two vectors a lane on either side of the numbers of
entries a row (4 fused, 12 for ragged FP32 SpMM on skewed columns) at which the
step of the run family changes: against the oracle, and the folded pass, whose step
does not change, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2404_19638_amd import synth
from test_gpu_run_family import DEV, Block, _np, _say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]


@pytest.mark.parametrize("kz,bf16", [(36, False), (60, False), (64, False), (72, True),
                                     (100, True), (128, True)])
@pytest.mark.parametrize("per_row,skew", [(4, False), (12, True), (12, False)])
@pytest.mark.parametrize("over", [0, 1])
def test_around_the_lines(kz, bf16, per_row, skew, over):
    n, cols_n = 1500, 4000
    rng = np.random.default_rng(per_row)
    at = lambda size: (rng.random(size) ** (6 if skew else 1) * cols_n).astype(np.int64)
    nnz = per_row * n - 1 + over
    rows = np.arange(nnz, dtype=np.int64) % n
    cols = at(nnz)
    while True:   # every (row, column) once
        keep = np.unique(rows * cols_n + cols, return_index=True)[1]
        again = np.setdiff1d(np.arange(nnz), keep)
        if again.size == 0:
            break
        cols[again] = rng.integers(0, cols_n, again.size)
    b = Block(rows, cols, n, cols_n)
    spc, plan = b.spc, b.plan
    assert plan.R == n and plan.nnz == nnz
    _say(f"run steps: nnz={nnz} kz={kz} bf16={bf16} skew={skew}")
    b.check(kz, bf16, what="run steps")
    _, _, Ad, Bd = b.operands(kz, bf16, 61)
    out, Y = spc.sddmm_spmm(plan, b.v, Ad, Bd, kz)
    slab0 = synth.dense_f32(9, 0, n, kz)
    after = slab0.copy()
    oracle.scatter_add_f32(b.ref["gmap_r"], 0, _np(Y), after, 0)
    slab = torch.from_numpy(slab0).to(DEV)
    out2 = spc.sddmm_spmm_scatter(plan, b.v, Ad, Bd, slab, 0, kz)
    np.testing.assert_array_equal(_np(slab).view(np.uint32), after.view(np.uint32))
    assert torch.equal(out2, out)
