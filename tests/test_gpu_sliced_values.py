"""Wide rows taken in slices by the fused pass: entries whose value times a
part of the dot overflows, or is infinite with another sign, while value times
the whole dot does not; in every output mode, with the slab's bits those of the
plain pass whatever out's mode is.  Also scratch smaller than the size asked
for.

Bars: |x - x*| <= 1e-5 M for finite x* (M the magnitude sum of the dot times
|value|, plus the accumulated output's one more rounding); infinities exact."""
import numpy as np
import pytest

import oracle
from paper_2404_19638_amd import synth
from test_gpu_run_family import DEV, Block, _np, _say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]

USED, N = 290_000, 1 << 20


@pytest.fixture(scope="module")
def block():
    r, c = synth.uniform_block(3000, USED, 1_200_000, 13)
    return Block(r, c * (N // USED), 3000, N)


@pytest.mark.parametrize("kz,bf16", [(128, False), (256, True), (160, False), (256, False)])
def test_values_times_parts_of_a_dot(block, kz, bf16):
    b, spc, plan = block, block.spc, block.plan
    _say(f"sliced values: kz={kz} bf16={bf16} nnz={plan.nnz}")
    dt = torch.bfloat16 if bf16 else torch.float32
    g = torch.Generator(device=DEV).manual_seed(3)
    x = torch.randint(1, 9, (plan.C, kz // 2), generator=g, device=DEV).float()
    A = torch.ones((plan.R, kz), device=DEV)
    # the two halves of a dot are near each other with opposite signs
    B = torch.cat([x, -x.flip(1)], 1)
    B[:, -1] += 0.5
    v = b.v.clone()
    v[0::7] = 3e38
    v[1::7] = -3e38
    v[2::7] = float("inf")
    A, B = A.to(dt), B.to(dt)
    rows = torch.repeat_interleave(torch.arange(plan.R, device=DEV),
                                   plan.maps()["rowptr"].diff().long())
    cols = plan.maps()["colidx"].long()
    want, mag = torch.empty(plan.nnz, dtype=torch.float64), torch.empty(plan.nnz)
    for i in range(0, plan.nnz, 1 << 18):   # in 64 bits, by parts of the entries
        p = A[rows[i:i + (1 << 18)]].double() * B[cols[i:i + (1 << 18)]].double()
        want[i:i + (1 << 18)] = (v[i:i + (1 << 18)].double() * p.sum(1)).cpu()
        mag[i:i + (1 << 18)] = p.abs().sum(1).float().cpu()
    want, mag = want.numpy(), mag.double().numpy()
    vmag = np.abs(_np(v).astype(np.float64))
    fits = np.abs(want) < 3.3e38
    inf = np.isinf(want)
    assert fits.sum() > plan.nnz // 2 and inf.sum() > plan.nnz // 8

    def check(out, out0, what):
        got = _np(out).astype(np.float64)
        assert (got[inf] == want[inf]).all(), what
        err = np.abs(got[fits] - np.add(out0, want)[fits])
        bar = (1e-5 * np.minimum(vmag * mag, 1e300) + 2.0 ** -23 * np.abs(out0))[fits]
        assert (err <= bar).all(), what

    buf = torch.empty(spc.spmm_buffer_size(plan, 0, kz), dtype=torch.uint8, device=DEV)
    out, Y = spc.sddmm_spmm(plan, v, A, B, kz, buf=buf)
    check(out, 0.0, "overwrite")
    o0 = synth.uniform_f32(7, plan.nnz)
    acc = torch.from_numpy(o0).to(DEV)
    spc.sddmm_spmm(plan, v, A, B, kz, out=acc, mode=spc.ACCUMULATE, buf=buf,
                   Y=torch.zeros_like(Y))
    check(acc, o0.astype(np.float64), "accumulate")
    # finite values for the rows: the slab holds their bits in both modes of out
    out, Y = spc.sddmm_spmm(plan, b.v, A, B, kz, buf=buf)
    slab0 = synth.dense_f32(9, 0, b.nr, kz + 4)
    want_slab = slab0.copy()
    oracle.scatter_add_f32(b.ref["gmap_r"], 0, _np(Y), want_slab, 4)
    for mode in (spc.OVERWRITE, spc.ACCUMULATE):
        slab = torch.from_numpy(slab0).to(DEV)
        o2 = torch.zeros_like(out)
        spc.sddmm_spmm_scatter(plan, b.v, A, B, slab, 4, kz, out=o2, out_mode=mode, buf=buf)
        np.testing.assert_array_equal(_np(slab).view(np.uint32), want_slab.view(np.uint32))


def test_no_values_and_less_scratch(block):
    b, spc, plan = block, block.spc, block.plan
    for kz, bf16 in ((128, False), (256, False)):
        A, B, Ad, Bd = b.operands(kz, bf16, 60)
        for vals, hv in ((None, np.ones_like(b.vals)), (b.v, b.vals)):
            o, mo = oracle.sddmm(b.rows, b.cols, 0, 0, hv, A, B, 0, kz)
            o, mo = o[b.ref["perm"]], mo[b.ref["perm"]]
            size = spc.spmm_buffer_size(plan, 0, kz)
            for n in (size, max(size - 4 * plan.nnz, size // 2), size // 2):
                _say(f"sliced scratch: kz={kz} {n} of {size}")
                buf = torch.empty(n, dtype=torch.uint8, device=DEV)
                o0 = synth.uniform_f32(7, plan.nnz)
                for mode, x0 in ((spc.OVERWRITE, 0.0), (spc.ACCUMULATE, o0.astype(np.float64))):
                    out = torch.from_numpy(o0).to(DEV)
                    try:
                        spc.sddmm_spmm(plan, vals, Ad, Bd, kz, out=out, mode=mode, buf=buf,
                                       Y=torch.zeros((plan.R, kz), device=DEV))
                    except spc.Spc3dError as e:
                        assert e.status == spc.ERR_WORKSPACE and n < size
                        continue
                    err = np.abs(_np(out).astype(np.float64) - (x0 + o))
                    assert (err <= 1e-5 * mo + 2.0 ** -23 * (np.abs(x0) + mo)).all(), (kz, n, mode)
