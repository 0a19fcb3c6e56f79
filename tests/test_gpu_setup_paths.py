"""Localization at the edges of its tiles: id ranges around the 64 ids of a
rank word, the 16384 of a block and of several blocks, entry counts around the
sort's tiles of 2048 and 4096 entries and its switch between them, one bit and
none of a key, and CSR rows that end at, inside and across the 512-entry
chunks of the row expansion (a row over many chunks, empty rows between)."""
import sys

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]

DEV = "cuda:0"
KEYS = ("gmap_r", "gmap_c", "rowptr", "colidx", "perm", "colptr", "rowidx_t", "slot_t")


def _compare(plan, rows, cols, rr, cr, what):
    print(f"setup: {what} nnz={rows.size}", file=sys.stderr, flush=True)
    ref = oracle.relabel(rows, cols, rr, cr, csc=True)
    m = plan.maps()
    for k in KEYS + ("lmap_r", "lmap_c"):
        np.testing.assert_array_equal(m[k].cpu().numpy(), ref[k], err_msg=f"{what} {k}")


def _coo(rows, cols, rr, cr, what):
    from paper_2404_19638_amd import spc3d as spc
    plan = spc.plan_create_coo(torch.from_numpy(rows).to(DEV), torch.from_numpy(cols).to(DEV), rr,
                               cr, spc.BUILD_CSC)
    spc.plan_check(plan)
    _compare(plan, rows, cols, rr, cr, what)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1000, 16383, 16384, 16385, 50001])
def test_id_ranges_around_words_and_blocks(n):
    rng = np.random.default_rng(n)
    lo = 7_000_000_001
    for m in (1, 3000):
        rows = rng.integers(0, n, m) + lo
        cols = rng.integers(0, 3 * n, m) - lo
        rows[0], cols[0] = lo + n - 1, 3 * n - 1 - lo   # the range's last ids
        _coo(rows, cols, (lo, lo + n), (-lo, 3 * n - lo), f"range {n}")


@pytest.mark.parametrize("nnz", [2047, 2048, 2049, 4097, (6 << 20) - 1, (6 << 20) + 1])
def test_entry_counts_around_sort_tiles(nnz):
    rng = np.random.default_rng(nnz)
    rows = rng.integers(0, 300_000, nnz) ** 2 // 300_000   # skewed, with duplicates
    cols = rng.integers(0, 70_000, nnz)
    _coo(rows, cols, (0, 300_000), (0, 70_000), f"tiles {nnz}")


@pytest.mark.parametrize("lengths", [[512], [511, 1, 512], [0, 0, 513, 0, 1], [3] * 400 + [0] * 90,
                                     [0] * 70 + [5000, 1, 0, 2] + [1] * 900, [0, 1] * 700])
def test_csr_rows_around_chunks(lengths):
    from paper_2404_19638_amd import spc3d as spc
    rng = np.random.default_rng(len(lengths))
    lengths = np.asarray(lengths, np.int64)
    ptr = np.concatenate([[0], np.cumsum(lengths)])
    cols = rng.integers(100, 6000, ptr[-1])
    plan = spc.plan_create_csr(torch.from_numpy(ptr).to(DEV), torch.from_numpy(cols).to(DEV),
                               (10, 10 + lengths.size), (100, 6000), spc.BUILD_CSC)
    rows = np.repeat(np.arange(lengths.size) + 10, lengths)
    _compare(plan, rows, cols, (10, 10 + lengths.size), (100, 6000), "csr")
