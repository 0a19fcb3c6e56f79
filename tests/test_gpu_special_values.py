"""Infinities, NaN and the lowest finite values through the kernels for ragged
rows and through the one-pass attention forward: each element is infinite or
NaN exactly where 64-bit arithmetic on the same operands makes it so, and what
a special value does not reach stays within the usual bar, |x - x*| <= 1e-5 M
(the attention's: 1e-5 of the row's largest |V| times its entries, at least)."""
import numpy as np
import pytest

from test_gpu_run_family import DEV, Block, _from_lengths, _lengths, _say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]

INF, NAN = float("inf"), float("nan")


def _structure(plan):
    m = plan.maps()
    ptr = m["rowptr"].long().cpu()
    rows = torch.repeat_interleave(torch.arange(plan.R), ptr.diff())
    return ptr, rows, m["colidx"].long().cpu()


def _same(got, want, mag, what):
    got = got.detach().double().cpu()
    assert torch.equal(got.isnan(), want.isnan()), what
    inf = want.isinf()
    assert torch.equal(got.isinf(), inf) and torch.equal(got[inf], want[inf]), what
    ok = want.isfinite()
    assert ((got - want).abs()[ok] <= 1e-5 * mag[ok]).all(), what


@pytest.mark.parametrize("kz,bf16", [(15, False), (30, False), (60, False), (127, False),
                                     (17, True), (30, True), (100, True), (250, True)])
def test_ragged_rows(kz, bf16):
    lengths = _lengths("mixed")
    b = Block(*_from_lengths(lengths, 2500, 4), len(lengths), 2500)
    spc, plan = b.spc, b.plan
    _say(f"special values: kz={kz} bf16={bf16}")
    g = torch.Generator().manual_seed(kz)
    dt = torch.bfloat16 if bf16 else torch.float32
    A, B = (torch.rand((n, kz), generator=g).sub(0.5).to(dt) for n in (plan.R, plan.C))
    v = torch.rand(plan.nnz, generator=g) - 0.5
    for X in (A, B):   # in the last vector, its overlap, and the first
        for i, (k, x) in enumerate(((kz - 1, INF), (kz - 8, -INF), (kz // 2, NAN), (0, INF))):
            X[3 + 17 * i, k] = x
    v[5::97] = 0.0     # times infinity: NaN
    v[7::101] = INF
    ptr, rows, cols = _structure(plan)
    Ad, Bd, vd = A.to(DEV), B.to(DEV), v.to(DEV)
    A64, B64 = A.double(), B.double()
    p = A64[rows] * B64[cols]
    dots, dmag = p.sum(1) * v.double(), p.abs().nan_to_num(0, 0, 0).sum(1) * v.abs().double()
    q = v.double()[:, None] * B64[cols]
    Y = torch.zeros((plan.R, kz), dtype=torch.float64).index_add_(0, rows, q)
    ymag = torch.zeros_like(Y).index_add_(0, rows, q.abs().nan_to_num(0, 0, 0))
    _same(spc.sddmm(plan, vd, Ad, Bd, kz), dots, dmag, f"sddmm {kz}")
    out, Yf = spc.sddmm_spmm(plan, vd, Ad, Bd, kz)
    _same(out, dots, dmag, f"fused sddmm {kz}")
    _same(Yf, Y, ymag, f"fused spmm {kz}")
    _same(spc.spmm(plan, vd, Bd, 0, kz), Y, ymag, f"spmm {kz}")
    slab = torch.zeros((b.nr, kz + 3), device=DEV)
    spc.sddmm_spmm_scatter(plan, vd, Ad, Bd, slab, 1, kz)
    rows_of = plan.maps()["gmap_r"].long()
    _same(slab[rows_of, 1:1 + kz], Y, ymag, f"folded {kz}")
    assert (slab[:, 0] == 0).all() and (slab[:, 1 + kz:] == 0).all()


@pytest.mark.parametrize("kz,bf16", [(16, False), (64, False), (128, False), (32, True),
                                     (64, True), (256, True)])
@pytest.mark.parametrize("lg_s", [None, 4, 6])
def test_attention_scores(kz, bf16, lg_s):
    """One column of K sets a score: Q is 1 there and 0 elsewhere, so that a
    score is that element of its K row."""
    lengths = _lengths("mixed")
    b = Block(*_from_lengths(lengths, 2500, 4), len(lengths), 2500)
    spc, plan = b.spc, b.plan
    variant = -1 if lg_s is None else 3 | (lg_s << 4)
    if variant >= 0 and not 8 <= kz * (2 if bf16 else 4) // 16 <= 16:
        variant = (2 if kz * (2 if bf16 else 4) == 64 else 4) | (lg_s << 4)
    _say(f"special scores: kz={kz} bf16={bf16} variant={variant}")
    dt = torch.bfloat16 if bf16 else torch.float32
    low = torch.finfo(dt).min
    g = torch.Generator().manual_seed(kz)
    score = torch.randn(plan.C, generator=g).mul(3)
    score[0::5] = -INF                # many rows have some, short ones may have no others
    score[1::50] = low
    score[2::211] = INF
    score[3::307] = NAN
    Q, K = torch.zeros((plan.R, kz)), torch.zeros((plan.C, kz))
    Q[:, 5], K[:, 5] = 1.0, score
    V = torch.rand((plan.C, kz), generator=g) - 0.5
    Q, K, V = Q.to(dt), K.to(dt), V.to(dt)
    ptr, rows, cols = _structure(plan)
    e = K[:, 5].double()[cols]
    # the row maximum among the scores that are numbers; equal scores weigh 1
    m = torch.full((plan.R,), -INF, dtype=torch.float64)
    m = m.scatter_reduce(0, rows, e.nan_to_num(-INF, INF, -INF), "amax")
    w = torch.where(e == m[rows], torch.ones_like(e), torch.exp(e - m[rows]))
    s = torch.zeros(plan.R, dtype=torch.float64).index_add_(0, rows, w)
    want = torch.zeros((plan.R, kz), dtype=torch.float64)
    want = want.index_add_(0, rows, w[:, None] * V.double()[cols]) / s[:, None]
    assert want.isnan().any() and want.isfinite().all(1).sum() > plan.R // 2
    out, _ = spc.attention_fwd(plan, Q.to(DEV), K.to(DEV), V.to(DEV), variant=variant)
    mag = torch.tensor(np.diff(ptr.numpy()), dtype=torch.float64)[:, None].clamp(min=8)
    _same(out, want, mag.expand_as(want), f"attention {kz}")
