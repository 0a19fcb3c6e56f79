"""gnn_attention's automatic forward choice by row width (no GPU needed): the
one pass on rows of up to 128 bytes at any size, wider ones up to a number of
entries that falls with the width."""
import types

import pytest

torch = pytest.importorskip("torch")
from paper_2404_19638_amd import autograd as ag, spc3d as spc   # noqa: E402


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("row_bytes", [64, 128, 256, 512])
def test_choice_by_row_width(dt, row_bytes):
    k = row_bytes // torch.empty(0, dtype=dt).element_size()
    qkv = [torch.zeros((8, k), dtype=dt) for _ in range(3)]
    code = spc.F32 if dt == torch.float32 else spc.BF16
    assert spc.attention_supported(k, code)
    limit = ag._AUTO_FUSED_MAX_NNZ.get((code, row_bytes))
    assert (limit is None) == (row_bytes <= 128)
    for nnz in (0, 1, 1 << 30) if limit is None else (0, 1, limit):
        assert ag._auto_fused(types.SimpleNamespace(nnz=nnz), *qkv)
    if limit is not None:
        assert not ag._auto_fused(types.SimpleNamespace(nnz=limit + 1), *qkv)
