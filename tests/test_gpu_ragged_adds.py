"""Rows added to what is there, at widths whose last vector is moved back over
its neighbour's elements (a bfloat16 lane holds two 16-byte halves of a row, and
the moved-back first half is another lane's second): every element gets the
plain pass's sum once, bit for bit, in Y and in a slab."""
import numpy as np
import pytest

import oracle
from paper_2404_19638_amd import synth
from test_gpu_run_family import DEV, Block, _from_lengths, _lengths, _np, _say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]


@pytest.mark.parametrize("kz,bf16", [(17, True), (20, True), (23, True), (41, True), (66, True),
                                     (132, True), (193, True), (9, False), (33, False),
                                     (66, False), (127, False)])
def test_overlapping_vectors_add_once(kz, bf16):
    lengths = _lengths("mixed")
    b = Block(*_from_lengths(lengths, 2500, 6), len(lengths), 2500)
    spc, plan = b.spc, b.plan
    _, _, Ad, Bd = b.operands(kz, bf16, 60)
    _say(f"ragged adds: kz={kz} bf16={bf16}")
    y0 = torch.from_numpy(synth.dense_f32(8, 0, plan.R, kz)).to(DEV)
    out, Y = spc.sddmm_spmm(plan, b.v, Ad, Bd, kz)
    Ys = spc.spmm(plan, b.v, Bd, 0, kz)
    Y2, Y3 = y0.clone(), y0.clone()
    spc.sddmm_spmm(plan, b.v, Ad, Bd, kz, out=torch.zeros_like(out), Y=Y2, mode=spc.ACCUMULATE)
    spc.spmm(plan, b.v, Bd, 0, kz, out=Y3, mode=spc.ACCUMULATE)
    assert torch.equal(Y2, y0 + Y)
    assert torch.equal(Y3, y0 + Ys)
    for ld, k0 in ((kz, 0), (kz + 8, 4), (kz + 6, 5)):
        dst0 = synth.dense_f32(9, 0, b.nr, ld)
        want = dst0.copy()
        oracle.scatter_add_f32(b.ref["gmap_r"], 0, _np(Y), want, k0)
        dst = torch.from_numpy(dst0).to(DEV)
        spc.sddmm_spmm_scatter(plan, b.v, Ad, Bd, dst, k0, kz)
        np.testing.assert_array_equal(_np(dst).view(np.uint32), want.view(np.uint32))
