"""Row pointers that plan creation refuses, over many more rows than entries:
the workspace lies inside a larger tensor, and what follows it stays as it was
(a row pointer that rises in every row marks more rows than the maps have room
for)."""
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]

DEV = "cuda:0"
ROWS = 1 << 20


def _rising(nnz):
    return torch.arange(ROWS + 1, device=DEV)


def _zigzag(nnz):
    """Inside [0, nnz], from 0 to nnz, rising in every other row."""
    p = (torch.arange(ROWS + 1, device=DEV) % 2) * nnz
    p[-1] = nnz
    return p


def _negative(nnz):
    p = torch.arange(ROWS + 1, device=DEV) - ROWS
    p[0], p[-1] = 0, nnz
    return p


@pytest.mark.parametrize("csc", [False, True])
@pytest.mark.parametrize("nnz", [0, 5, 2049])
@pytest.mark.parametrize("pointer", [_rising, _zigzag, _negative])
def test_refused_pointer_stays_in_its_workspace(pointer, nnz, csc):
    from paper_2404_19638_amd import spc3d as spc
    print(f"csr refused: {pointer.__name__} nnz={nnz} csc={csc}", file=sys.stderr, flush=True)
    rowptr = pointer(nnz)
    if nnz == 0 and pointer is _zigzag:
        rowptr = rowptr + torch.arange(ROWS + 1, device=DEV) % 2   # 0, 1, 0, 1, ... 0
        rowptr[-1] = 0
    cols = torch.arange(nnz, device=DEV) % 10
    flags = spc.BUILD_CSC if csc else 0
    need = spc.plan_workspace_size(nnz, 0, ROWS, 0, 10, flags)
    # room for a map entry per row twice over
    room = torch.full((need + 16 * ROWS,), 0xA5, dtype=torch.uint8, device=DEV)
    with pytest.raises(spc.Spc3dError) as ei:
        spc.plan_create_csr(rowptr, cols, (0, ROWS), (0, 10), flags, ws=room[:need])
    assert ei.value.status == spc.ERR_INVALID_ARG
    assert bool((room[need:] == 0xA5).all())
