"""The one-pass attention forward on a block of more than 2^24 rows and
columns, where row offsets take 64 bits: with one entry per row each output
row is its value row exactly, whatever the score; and blocks that end around
the ends of runs and work items, against the FP64 oracle within the bound that
test_gpu_attention_fused.py derives."""
import sys

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]

DEV = "cuda:0"


@pytest.mark.parametrize("dtype,kz", [(torch.bfloat16, 32), (torch.float32, 16)])
def test_more_rows_than_24_bits(dtype, kz):
    from paper_2404_19638_amd import spc3d as spc
    n = (1 << 24) + 77
    print(f"attention: n={n} kz={kz} {dtype}", file=sys.stderr, flush=True)
    rows = torch.arange(n, device=DEV)
    plan = spc.plan_create_coo(rows, n - 1 - rows, (0, n), (0, n))
    g = torch.Generator(device=DEV).manual_seed(3)
    Q, K, V = (torch.empty((n, kz), device=DEV).uniform_(-1, 1, generator=g).to(dtype)
               for _ in range(3))
    out, stats = spc.attention_fwd(plan, Q, K, V)
    assert torch.equal(out, V.float().flip(0))
    assert torch.equal(stats[:, 1], torch.ones(n, device=DEV))


@pytest.mark.parametrize("lg_s", [4, 5, 6])
@pytest.mark.parametrize("dtype,kz,lg_lanes", [(torch.float32, 64, 4), (torch.bfloat16, 64, 3),
                                               (torch.float32, 16, 2), (torch.bfloat16, 256, 4)])
def test_items_that_end_anywhere(dtype, kz, lg_lanes, lg_s):
    """Entry counts around the ends of runs and work items, rows of 1 to 7
    entries in turn so that rows start at every slot of a step."""
    import test_gpu_attention_fused as fused
    spc = fused._spc()
    run, item = 1 << lg_s, (64 >> lg_lanes) << lg_s
    for nnz in sorted({1, run - 1, run, run + 1, item - 1, item, item + 1, 2 * item + 3}):
        lengths = np.resize(np.arange(1, 8), nnz)
        rows = np.repeat(np.arange(nnz), lengths)[:nnz]
        cols = np.arange(nnz, dtype=np.int64)
        R = int(rows[-1]) + 1
        print(f"attention: nnz={nnz} kz={kz} {dtype} lg_s={lg_s}", file=sys.stderr, flush=True)
        plan = spc.plan_create_coo(torch.from_numpy(rows).to(DEV), torch.from_numpy(cols).to(DEV),
                                   (0, R), (0, nnz))
        rng = np.random.default_rng(100 * lg_s + nnz)
        Q, K, V = (rng.uniform(-1, 1, (n, kz)).astype(np.float32)
                   for n in (plan.R, plan.C, plan.C))
        rounded = [torch.from_numpy(x).to(dtype).float().numpy() for x in (Q, K, V)]
        ref = oracle.relabel(rows, cols, (0, R), (0, nnz))
        fused._check(spc, plan, ref, Q, K, V, kz, dtype, lg_lanes | lg_s << 4,
                     f"{dtype} kz={kz} nnz={nnz}", rounded)


@pytest.mark.parametrize("lg_s", [4, 5, 6])
def test_a_smaller_buffer_takes_longer_runs(lg_s):
    """The automatic shape with a buffer of an explicit run length's size gives
    that run length's result; one byte less than the longest's is refused."""
    from paper_2404_19638_amd import spc3d as spc
    n, kz = 3000, 64
    key = torch.arange(0, n * n, 601, device=DEV)
    plan = spc.plan_create_coo(key // n, key % n, (0, n), (0, n))
    g = torch.Generator(device=DEV).manual_seed(5)
    Q, K, V = (torch.rand((r, kz), device=DEV, generator=g) for r in (plan.R, plan.C, plan.C))
    v = 4 | lg_s << 4
    size = spc.attention_fwd_buffer_size(plan, kz, spc.F32, v)
    buf = torch.empty(size, dtype=torch.uint8, device=DEV)
    print(f"attention: nnz={plan.nnz} buffer={size}", file=sys.stderr, flush=True)
    want, _ = spc.attention_fwd(plan, Q, K, V, variant=v)
    got, _ = spc.attention_fwd(plan, Q, K, V, buf=buf)
    assert torch.equal(got, want)
    if lg_s == 6:
        with pytest.raises(spc.Spc3dError) as e:
            spc.attention_fwd(plan, Q, K, V, buf=buf[:size - 1])
        assert e.value.status == spc.ERR_WORKSPACE
