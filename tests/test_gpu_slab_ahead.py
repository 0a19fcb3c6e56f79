"""Rows of one to five entries added to a slab of 48 MB and more (whose rows the
pass reads where a row starts) and just below: the slab ends bit for bit as the
plain pass's rows added to it."""
import numpy as np
import pytest

import oracle
from paper_2404_19638_amd import synth
from test_gpu_run_family import DEV, Block, _np, _say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]


@pytest.mark.parametrize("kz,bf16", [(16, False), (32, False), (64, False), (32, True), (64, True)])
@pytest.mark.parametrize("over", [0, 1])
def test_short_rows_into_a_large_slab(kz, bf16, over):
    n = (48 << 20) // (4 * kz) - 1 + over
    rng = np.random.default_rng(kz)
    lengths = rng.integers(1, 5, n)
    lengths[rng.integers(0, n, n // 3)] = 1
    rows = np.repeat(np.arange(n, dtype=np.int64), lengths)
    cols = (rows * 7 + np.arange(rows.size) * 13) % 2000
    keep = np.unique(rows * 2000 + cols, return_index=True)[1]
    b = Block(rows[keep], cols[keep], n, 2000)
    spc, plan = b.spc, b.plan
    assert plan.R == n and plan.nnz < 3 * n
    _say(f"slab ahead: R={n} nnz={plan.nnz} kz={kz} bf16={bf16}")
    _, _, Ad, Bd = b.operands(kz, bf16, 60)
    out, Y = spc.sddmm_spmm(plan, b.v, Ad, Bd, kz)
    slab0 = synth.dense_f32(9, 0, n, kz)
    want = slab0.copy()
    oracle.scatter_add_f32(b.ref["gmap_r"], 0, _np(Y), want, 0)
    slab = torch.from_numpy(slab0).to(DEV)
    out2 = spc.sddmm_spmm_scatter(plan, b.v, Ad, Bd, slab, 0, kz)
    np.testing.assert_array_equal(_np(slab).view(np.uint32), want.view(np.uint32))
    assert torch.equal(out2, out)
