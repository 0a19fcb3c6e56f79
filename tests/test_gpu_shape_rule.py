"""SpMM and the fused pass on either side of the lines between the run family
and the other shapes: blocks above 2^17 entries with equal rows around 5, 10 and
20 entries, wide rows, aligned and misaligned operands, in buffers of exactly
the size asked for, against the FP64 oracle.

Bar: |x - x*| <= 1e-5 M, M the oracle's magnitude sum, as in
test_gpu_run_family.py, whose Block draws the inputs."""
import pytest

import oracle
from helpers import assert_within_mag
from test_gpu_run_family import DEV, Block, _from_lengths, _np, _say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]


@pytest.mark.parametrize("per_row", [4, 5, 9, 10, 19, 20])
def test_wide_rows_around_the_lines(per_row):
    nr = 132_000 // per_row
    b = Block(*_from_lengths([per_row] * nr, 30_000, 17), nr, 30_000)
    spc, plan, ref = b.spc, b.plan, b.ref
    for kz, bf16, shift in ((128, False, 0), (128, False, 1), (96, False, 0), (128, True, 0)):
        A, B, Ad, Bd = b.operands(kz, bf16, 60, shift)
        o, mo = oracle.sddmm(b.rows, b.cols, 0, 0, b.vals, A, B, 0, kz)
        y, my = oracle.spmm(b.rows, b.cols, 0, 0, ref["lmap_r"], ref["R"], b.vals, B, 0, kz)
        _say(f"shape rule: per_row={per_row} nnz={plan.nnz} kz={kz} bf16={bf16} shift={shift}")
        buf = torch.empty(spc.spmm_buffer_size(plan, 0, kz), dtype=torch.uint8, device=DEV)
        out, Y = spc.sddmm_spmm(plan, b.v, Ad, Bd, kz, buf=buf)
        assert_within_mag(_np(out), o[ref["perm"]], mo[ref["perm"]], what=f"sddmm {per_row} {kz}")
        assert_within_mag(_np(Y), y, my, what=f"fused spmm {per_row} {kz}")
        Ys = spc.spmm(plan, b.v, Bd, 0, kz, buf=buf)
        assert_within_mag(_np(Ys), y, my, what=f"spmm {per_row} {kz}")
        for ld, k0 in ((kz + 4, 4), (kz + 5, 3)):   # an aligned slab and one that is not
            dst = torch.zeros((b.nr, ld), device=DEV)
            spc.sddmm_spmm_scatter(plan, b.v, Ad, Bd, dst, k0, kz, buf=buf)
            got = _np(dst)[ref["gmap_r"], k0:k0 + kz]
            assert_within_mag(got, y, my, what=f"folded {per_row} {kz} ld={ld}")
