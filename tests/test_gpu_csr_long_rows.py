"""CSR rows over many of the row expansion's 512-entry chunks: around the 8
chunks from which a wavefront marks a row together, several such rows among its
64, one row over hundreds of chunks, and the last row of the range."""
import numpy as np
import pytest

from test_gpu_setup_paths import DEV, _compare

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]

C = 512


@pytest.mark.parametrize("lengths", [[8 * C], [8 * C + 1], [9 * C], [1, 9 * C - 1, 9 * C + 1],
                                     [3] * 62 + [20 * C, 0, 64 * C + 7, 2], [0] * 130 + [200_000],
                                     [1, 300 * C + 3, 0] + [5] * 100 + [40 * C] * 5])
def test_rows_over_many_chunks(lengths):
    from paper_2404_19638_amd import spc3d as spc
    rng = np.random.default_rng(len(lengths))
    lengths = np.asarray(lengths, np.int64)
    ptr = np.concatenate([[0], np.cumsum(lengths)])
    cols = rng.integers(0, 30_000, ptr[-1])
    plan = spc.plan_create_csr(torch.from_numpy(ptr).to(DEV), torch.from_numpy(cols).to(DEV),
                               (7, 7 + lengths.size), (0, 30_000), spc.BUILD_CSC)
    rows = np.repeat(np.arange(lengths.size) + 7, lengths)
    _compare(plan, rows, cols, (7, 7 + lengths.size), (0, 30_000), "long rows")
