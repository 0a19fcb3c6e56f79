"""The order in which a row is summed follows from the operands, not from where
the row goes: a slab of any ld and k0, and a Y at any address, hold the bits of
the plain pass, on blocks small and large, short rows and long, in the default
shape and in explicit ones."""
import numpy as np
import pytest

import oracle
from paper_2404_19638_amd import synth
from test_gpu_run_family import DEV, Block, _from_lengths, _np, _say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]

GROUP_RUNS, WINDOWS = 3 | (3 << 4), 3 | (1 << 4) | (1 << 9)   # 8 lanes, items of 512 and 128


def _check(b, kz, bf16, variant=-1):
    spc, plan = b.spc, b.plan
    _, _, Ad, Bd = b.operands(kz, bf16, 60)
    _say(f"slab bits: nnz={plan.nnz} R={plan.R} kz={kz} bf16={bf16} variant={variant}")
    out, Y = spc.sddmm_spmm(plan, b.v, Ad, Bd, kz, variant=variant)
    Ys = spc.spmm(plan, b.v, Bd, 0, kz, variant=variant)
    for at in (1, 2):
        buf = torch.empty(plan.R * kz + at, device=DEV)
        Yu = buf[at:].view(plan.R, kz)
        out2, _ = spc.sddmm_spmm(plan, b.v, Ad, Bd, kz, Y=Yu, variant=variant)
        assert torch.equal(Yu, Y) and torch.equal(out2, out), (kz, at)
        spc.spmm(plan, b.v, Bd, 0, kz, out=Yu, variant=variant)
        assert torch.equal(Yu, Ys), (kz, at)
    for ld, k0 in ((kz + 4, 4), (kz + 4, 1), (kz + 5, 4), (kz + 5, 3)):
        dst0 = synth.dense_f32(9, 0, b.nr, ld)
        want = dst0.copy()
        oracle.scatter_add_f32(b.ref["gmap_r"], 0, _np(Y), want, k0)
        dst = torch.from_numpy(dst0).to(DEV)
        out3 = spc.sddmm_spmm_scatter(plan, b.v, Ad, Bd, dst, k0, kz, variant=variant)
        np.testing.assert_array_equal(_np(dst).view(np.uint32), want.view(np.uint32),
                                      err_msg=f"kz={kz} ld={ld} k0={k0}")
        assert torch.equal(out3, out), (kz, ld, k0)


@pytest.mark.parametrize("entries,per_row", [(3000, 5), (140_000, 4), (140_000, 12),
                                             (300_000, 30), (1_100_000, 6)])
def test_default_shape(entries, per_row):
    nr = entries // per_row
    b = Block(*_from_lengths([per_row] * nr, 2000, 18), nr, 2000)
    for kz, bf16 in ((4, False), (8, False), (32, False), (96, False), (128, False),
                     (8, True), (16, True), (128, True)):
        _check(b, kz, bf16)


def test_more_than_512_bytes_a_row():
    b = Block(*_from_lengths([3, 90, 1, 17, 400] * 30, 2000, 19), 150, 2000)
    for kz, bf16 in ((200, False), (256, False), (256, True)):
        _check(b, kz, bf16)


@pytest.mark.parametrize("variant", [GROUP_RUNS, WINDOWS])
def test_explicit_shape(variant):
    b = Block(*_from_lengths([3, 90, 1, 17, 400] * 60, 2000, 20), 300, 2000)
    # (rows of more than 32 values in 8 lanes are refused off alignment, as before)
    for kz, bf16 in ((20, False), (32, False), (24, True)):
        _check(b, kz, bf16, variant)


def test_refused_destinations_stay_refused():
    """Rows beyond the widest scalar shape need an aligned destination."""
    from paper_2404_19638_amd import spc3d as spc
    b = Block(*_from_lengths([3, 9, 1], 200, 21), 3, 200)
    kz = 260
    _, _, Ad, Bd = b.operands(kz, False, 60)
    spc.sddmm_spmm_scatter(b.plan, b.v, Ad, Bd, torch.zeros((3, kz + 4), device=DEV), 4, kz)
    for ld, k0 in ((kz + 5, 4), (kz + 4, 1)):
        with pytest.raises(spc.Spc3dError) as ei:
            spc.sddmm_spmm_scatter(b.plan, b.v, Ad, Bd, torch.zeros((3, ld), device=DEV), k0, kz)
        assert ei.value.status == spc.ERR_UNSUPPORTED
