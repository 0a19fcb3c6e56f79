"""Both sides of the lines at which wide rows go from the run family to the other
shapes: bfloat16 rows of two and four vectors a lane, on columns used evenly and
not, and rows of 512 bytes and more taken in slices from a number of entries a
row; element by element against the FP64 oracle, the folded slab bit for bit
(Block.check of test_gpu_run_family.py)."""
import pytest

from paper_2404_19638_amd import synth
from test_gpu_run_family import Block

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]


@pytest.mark.parametrize("nnz,kz", [((1 << 17) - 1, 256), (1 << 17, 256), ((1 << 19) - 1, 96),
                                    (1 << 19, 96), (1 << 20, 96)])
@pytest.mark.parametrize("skew", [1, 5])   # every column of the range, or one in five
def test_bfloat16_rows(nnz, kz, skew):
    r, c = synth.uniform_block(20_000, 10_000, nnz, 31)
    b = Block(r, c * skew, 20_000, 10_000 * skew)
    b.check(kz, True, what=f"lines, skew {skew}")


@pytest.mark.parametrize("kz,bf16,per_row", [(128, False, 35), (128, False, 37), (256, True, 35),
                                             (256, True, 37), (192, False, 27),
                                             (192, False, 29)])
def test_rows_in_slices(kz, bf16, per_row):
    n, used, nnz = 1 << 20, 290_000, 1_200_000
    rows = nnz // per_row
    r, c = synth.uniform_block(rows, used, nnz, 13)
    b = Block(r, c * (n // used), rows, n)
    b.check(kz, bf16, what=f"slices from {per_row} entries")
