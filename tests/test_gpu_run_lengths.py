"""SpMM and the fused pass at every length of the run family's runs: blocks on
both sides of the numbers of entries at which the default takes runs of 8, 16
and 32 slots (groups of 4 and of 8 lanes), with rows that end anywhere and a row
over many items, element by element against the FP64 oracle.  Bars as in
test_gpu_run_family.py."""
import numpy as np
import pytest

from test_gpu_run_family import Block, _from_lengths

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]


def _block(nnz, most):
    """nnz entries in rows of 1 to most entries, one of 1500 among them."""
    rng = np.random.default_rng(nnz + most)
    lengths = [1500]
    left = nnz - 1500
    draws = rng.integers(1, most + 1, left)
    ends = np.searchsorted(np.cumsum(draws), left)
    lengths = list(draws[:ends // 2]) + lengths + list(draws[ends // 2:ends])
    lengths.append(nnz - sum(lengths))
    b = Block(*_from_lengths([n for n in lengths if n > 0], 2000, 23), len(lengths), 2000)
    assert b.plan.nnz == nnz
    return b


# 8 lanes: 64 * 1000, 128 * 1800, 128 * 2500 entries; 4 lanes: 128 * 1500, 256 * 4000
@pytest.mark.parametrize("nnz", [63_999, 64_000, 191_999, 192_000, 230_399, 230_400, 319_999,
                                 320_000])
def test_around_the_lines(nnz):
    b = _block(nnz, 12)
    for kz, bf16 in ((16, False), (30, False), (64, False), (24, True), (100, True)):
        b.check(kz, bf16, what="run lengths")


@pytest.mark.parametrize("nnz", [1_023_999, 1_024_000])
def test_around_the_last_line_of_four_lanes(nnz):
    b = _block(nnz, 40)
    b.check(16, False, what="run lengths")
    b.check(32, True, what="run lengths")
