"""The attention layer as one autograd function against the three functions it
is made of, and the softmax backward that also leaves alpha and de in column
order against the backward and two permutations: the same kernels' arithmetic
in the same order, so bit for bit."""
import itertools
import sys

import pytest

from paper_2404_19638_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]

DEV = "cuda:0"


def _plan(spc, n, nnz, flags):
    r, c = synth.uniform_block(n, n, nnz, 31 + nnz)
    return spc.plan_create_coo(torch.from_numpy(r).to(DEV), torch.from_numpy(c).to(DEV),
                               (0, n), (0, n), flags)


@pytest.mark.parametrize("n,nnz", [(1, 1), (40, 63), (40, 64), (40, 65), (300, 511), (300, 513),
                                   (300, 1025), (2000, 70_001)])
def test_columns_equal_backward_and_two_permutations(n, nnz):
    from paper_2404_19638_amd import spc3d as spc
    plan = _plan(spc, n, nnz, spc.BUILD_CSC)
    print(f"softmax columns: n={n} nnz={plan.nnz}", file=sys.stderr, flush=True)
    g = torch.Generator(device=DEV).manual_seed(nnz)
    alpha, dalpha = (torch.rand(plan.nnz, device=DEV, generator=g) for _ in range(2))
    de = spc.row_softmax_bwd(plan, alpha, dalpha)
    got, alpha_t, de_t = spc.row_softmax_bwd_columns(plan, alpha, dalpha.clone())
    assert torch.equal(got, de)
    assert torch.equal(alpha_t, spc.permute_values(plan, spc.SLOT_TO_COLUMN, alpha))
    assert torch.equal(de_t, spc.permute_values(plan, spc.SLOT_TO_COLUMN, de))
    place = dalpha.clone()
    spc.row_softmax_bwd_columns(plan, alpha, place, out=place)
    assert torch.equal(place, de)


def test_columns_need_the_column_view():
    from paper_2404_19638_amd import spc3d as spc
    plan = _plan(spc, 40, 64, 0)
    x = torch.rand(plan.nnz, device=DEV)
    with pytest.raises(spc.Spc3dError):
        spc.row_softmax_bwd_columns(plan, x, x.clone())


@pytest.mark.parametrize("limit", [0, 1 << 22])
@pytest.mark.parametrize("qk,v", [(torch.float32, torch.float32), (torch.bfloat16, torch.bfloat16),
                                  (torch.float32, torch.bfloat16)])
def test_layer_equals_its_three_functions(limit, qk, v, monkeypatch):
    from paper_2404_19638_amd import autograd as ag, spc3d as spc
    monkeypatch.setattr(ag, "DIRECT_MAX_NNZ", limit)
    plan = _plan(spc, 500, 6000, spc.BUILD_CSC)
    g = torch.Generator(device=DEV).manual_seed(7)
    kz = 40
    base = [torch.rand((r, kz), device=DEV, generator=g).to(t)
            for r, t in ((plan.R, qk), (plan.C, qk), (plan.C, v))]
    dout = torch.rand((kz, plan.R), device=DEV, generator=g).t()   # not contiguous
    for needs in itertools.product((False, True), repeat=3):
        if not any(needs):
            continue
        print(f"layer: limit={limit} {qk} {v} needs={needs}", file=sys.stderr, flush=True)
        grads = []
        for one in (True, False):
            Q, Kf, V = (x.clone().requires_grad_(n) for x, n in zip(base, needs))
            if one:
                out = ag.gnn_attention(plan, Q, Kf, V, fused=False)
            else:
                out = ag.spmm(plan, ag.row_softmax(plan, ag.sddmm(plan, None, Q, Kf)), V)
            wanted = [x for x, n in zip((Q, Kf, V), needs) if n]
            twice = [torch.autograd.grad(out, wanted, dout, retain_graph=True) for _ in range(2)]
            grads.append([out.detach(), *twice[0], *twice[1]])
        assert len(grads[0]) == len(grads[1])
        for x, y in zip(*grads):
            assert x.dtype == y.dtype and torch.equal(x, y), needs
