"""SDDMM on ragged bfloat16 rows: widths around every lane count, odd ones that
keep the element loads beside them, offset operands, both modes, against the
FP64 oracle's dots of the same bfloat16 values.

Tolerance: a length-kz FP32 dot of exact products, times v, added into out:
|error| <= (kz + 4) u M with M = |out before| + |v| sum_k |a_k b_k|, u = 2^-24."""
import sys

import numpy as np
import pytest

import oracle
from paper_2404_19638_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]

DEV = "cuda:0"
U = 2.0 ** -24


@pytest.mark.parametrize("kz", [7, 8, 9, 10, 14, 16, 18, 30, 31, 34, 62, 64, 66, 126, 130, 250, 254])
@pytest.mark.parametrize("offset", [0, 1, 2])
def test_ragged_widths(kz, offset):
    from paper_2404_19638_amd import spc3d as spc
    n = 300
    for nnz in (1, 63, 65, 2000):
        r, c = synth.uniform_block(n, n, nnz, 11 + nnz)
        ref = oracle.relabel(r, c, (0, n), (0, n))
        plan = spc.plan_create_coo(torch.from_numpy(r).to(DEV), torch.from_numpy(c).to(DEV),
                                   (0, n), (0, n))
        print(f"sddmm: kz={kz} offset={offset} nnz={plan.nnz}", file=sys.stderr, flush=True)
        ops = []
        for seed, rows in ((1, plan.R), (2, plan.C)):
            flat = torch.empty(offset + rows * kz, dtype=torch.bfloat16, device=DEV)
            x = torch.from_numpy(synth.dense_f32(seed, 0, rows, kz)).to(DEV).to(torch.bfloat16)
            flat[offset:] = x.flatten()
            ops.append(flat[offset:].view(rows, kz))
        A, B = ops
        Ad, Bd = (t.float().cpu().numpy().astype(np.float64) for t in (A, B))
        lr = np.repeat(np.arange(plan.R), np.diff(ref["rowptr"]))
        prod = Ad[lr] * Bd[ref["colidx"]]
        v = synth.dense_f32(3, 0, plan.nnz, 1).ravel()
        for vals in (None, v):
            w = np.ones(plan.nnz) if vals is None else vals.astype(np.float64)
            tv = None if vals is None else torch.from_numpy(vals).to(DEV)
            before = torch.from_numpy(synth.dense_f32(4, 0, plan.nnz, 1).ravel()).to(DEV)
            for mode in (spc.OVERWRITE, spc.ACCUMULATE):
                out = before.clone()
                spc.sddmm(plan, tv, A, B, out=out, mode=mode)
                old = before.cpu().numpy().astype(np.float64) * (mode == spc.ACCUMULATE)
                bar = (kz + 4) * U * (np.abs(old) + np.abs(w) * np.abs(prod).sum(1))
                err = np.abs(out.cpu().numpy() - (old + w * prod.sum(1)))
                assert np.all(err <= bar), (kz, offset, nnz, mode, float((err - bar).max()))
