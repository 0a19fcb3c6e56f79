"""The run family of the SpMM and fused kernels (the default shape of rows of
3 to 32 16-byte vectors), element by element against the FP64 oracle: work
items and runs that end inside rows, rows over many items, one entry, widths
that are not a multiple of a vector, misaligned operands, every output mode,
runs of each length, and slices of wide rows on blocks with skewed columns.

Bars: |x - x*| <= 1e-5 M, M the oracle's magnitude sum (bfloat16 operands
against the oracle on the same rounded values); an accumulated output adds
2^-23 (|x0| + M) for its one more rounding; the folded slab bit for bit as the
plain pass's rows added in FP32."""
import sys

import numpy as np
import pytest

import oracle
from paper_2404_19638_amd import synth
from helpers import assert_within_mag

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():   # pragma: no cover
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]

DEV = "cuda:0"


def _say(*a):
    print(*a, file=sys.stderr, flush=True)


def _np(t):
    return t.detach().float().cpu().numpy()


def _from_lengths(lengths, ncols, seed):
    """Rows of the given lengths with distinct columns, in row order."""
    rng = np.random.default_rng(seed)
    rows = np.repeat(np.arange(len(lengths), dtype=np.int64), lengths)
    cols = np.concatenate([rng.choice(ncols, n, replace=False) for n in lengths])
    return rows, cols.astype(np.int64)


def _lengths(name):
    rng = np.random.default_rng(5)
    return {
        "one entry": [1],
        "63 entries": [20, 1, 42],
        "one item": [64, 1, 63],             # 8 groups of 16 slots
        "one item and one": [100, 29],
        "a row over many items": [3, 1700, 2, 1, 900, 5],
        "all rows of one entry": [1] * 777,
        "mixed": list(rng.integers(1, 40, 300)) + [600] + list(rng.integers(1, 4, 200)),
    }[name]


class Block:
    def __init__(self, rows, cols, nr, nc, flags=0):
        from paper_2404_19638_amd import spc3d as spc
        self.spc, self.rows, self.cols, self.nr, self.nc = spc, rows, cols, nr, nc
        self.ref = oracle.relabel(rows, cols, (0, nr), (0, nc))
        self.plan = spc.plan_create_coo(torch.from_numpy(rows).to(DEV),
                                        torch.from_numpy(cols).to(DEV), (0, nr), (0, nc), flags)
        self.vals = synth.uniform_f32(41, rows.shape[0])
        self.v = torch.from_numpy(self.vals[self.ref["perm"]]).to(DEV)

    def operands(self, kz, bf16, seed, shift=0):
        """Host A, B over the id ranges and the packed device operands, `shift`
        elements past an aligned address."""
        A, B = synth.dense_f32(seed, 0, self.nr, kz), synth.dense_f32(seed + 1, 0, self.nc, kz)
        if bf16:
            A, B = (oracle.bf16_to_f32(oracle.bf16_rne(x)) for x in (A, B))
        dev = []
        for x, g in ((A, "gmap_r"), (B, "gmap_c")):
            p = torch.from_numpy(np.ascontiguousarray(x[self.ref[g]])).to(DEV)
            p = p.bfloat16() if bf16 else p
            buf = torch.empty(p.numel() + shift, dtype=p.dtype, device=DEV)
            buf[shift:] = p.reshape(-1)
            dev.append(buf[shift:].view(p.shape))
        return A, B, dev[0], dev[1]

    def check(self, kz, bf16, seed=60, shift=0, vals=True, what=""):
        spc, plan, ref = self.spc, self.plan, self.ref
        A, B, Ad, Bd = self.operands(kz, bf16, seed, shift)
        v = self.v if vals else None
        hv = self.vals if vals else np.ones_like(self.vals)
        o, mo = oracle.sddmm(self.rows, self.cols, 0, 0, hv, A, B, 0, kz)
        y, my = oracle.spmm(self.rows, self.cols, 0, 0, ref["lmap_r"], ref["R"], hv, B, 0, kz)
        o, mo = o[ref["perm"]], mo[ref["perm"]]
        _say(f"run family: {what} nnz={plan.nnz} kz={kz} bf16={bf16} shift={shift}")
        out, Y = spc.sddmm_spmm(plan, v, Ad, Bd, kz)
        assert_within_mag(_np(out), o, mo, what=f"sddmm {what} kz={kz}")
        assert_within_mag(_np(Y), y, my, what=f"fused spmm {what} kz={kz}")
        Ys = spc.spmm(plan, v, Bd, 0, kz)
        assert_within_mag(_np(Ys), y, my, what=f"spmm {what} kz={kz}")
        # accumulated into prefilled outputs
        o0 = torch.from_numpy(synth.uniform_f32(7, plan.nnz)).to(DEV)
        y0 = torch.from_numpy(synth.dense_f32(8, 0, plan.R, kz)).to(DEV)
        out2, Y2 = o0.clone(), y0.clone()
        spc.sddmm_spmm(plan, v, Ad, Bd, kz, out=out2, Y=Y2, mode=spc.ACCUMULATE)
        for got, x0, x, m in ((out2, o0, o, mo), (Y2, y0, y, my)):
            err = np.abs(_np(got).astype(np.float64) - (_np(x0).astype(np.float64) + x))
            assert (err <= 1e-5 * m + 2.0 ** -23 * (np.abs(_np(x0)) + m)).all(), f"{what} {kz}"
        # the folded slab: one FP32 addition of the plain pass's rows
        dst0 = synth.dense_f32(9, 0, self.nr, kz + 5)
        want = dst0.copy()
        oracle.scatter_add_f32(ref["gmap_r"], 0, _np(Y), want, 3)
        dst = torch.from_numpy(dst0).to(DEV)
        out3 = spc.sddmm_spmm_scatter(plan, v, Ad, Bd, dst, 3, kz)
        np.testing.assert_array_equal(_np(dst).view(np.uint32), want.view(np.uint32))
        assert torch.equal(out3, out)


@pytest.mark.parametrize("name", ["one entry", "63 entries", "one item", "one item and one",
                                  "a row over many items", "all rows of one entry", "mixed"])
def test_runs_and_items_that_end_inside_rows(name):
    lengths = _lengths(name)
    b = Block(*_from_lengths(lengths, 2500, 3), len(lengths), 2500)
    for kz, bf16 in ((16, False), (32, False), (64, False), (128, False), (64, True), (256, True)):
        b.check(kz, bf16, what=name)
    b.check(32, False, vals=False, what=name + ", no values")


@pytest.mark.parametrize("kz,bf16", [(9, False), (15, False), (17, False), (30, False), (33, False),
                                     (60, False), (67, False), (120, False), (127, False),
                                     (17, True), (30, True), (65, True), (120, True), (251, True)])
def test_widths_between_vectors_and_misaligned_operands(kz, bf16):
    lengths = _lengths("mixed")
    b = Block(*_from_lengths(lengths, 2500, 4), len(lengths), 2500)
    b.check(kz, bf16, what="mixed")
    b.check(kz, bf16, shift=1, what="mixed, shifted")


@pytest.mark.parametrize("rows,nnz", [(60_000, 1_900_000), (120_000, 3_800_000)])
def test_runs_of_32_and_64_slots(rows, nnz):
    """Long rows (over 16 entries) on blocks large enough for the longer runs."""
    r, c = synth.uniform_block(rows, 50_000, nnz, 11)
    b = Block(r, c, rows, 50_000)
    for kz in (16, 30, 64):
        b.check(kz, False, what="long runs")


@pytest.mark.parametrize("used,kz,bf16", [(110_000, 128, False), (290_000, 128, False),
                                          (290_000, 64, False), (290_000, 128, True),
                                          (380_000, 96, False)])
def test_slices_of_wide_rows_on_skewed_columns(used, kz, bf16):
    """Columns from a part of the id range (a block whose entries share columns
    takes wide rows in slices), also transposed."""
    n = 1 << 20
    r, c = synth.uniform_block(3000, used, 1_200_000, 13)
    b = Block(r, c * (n // used), 3000, n)
    b.check(kz, bf16, what=f"slices, {used} columns")
    # the transposed product gathers the table whose rows are spread likewise
    from paper_2404_19638_amd import spc3d as spc
    bt = Block(c * (n // used), r, n, 3000, spc.BUILD_CSC)
    X = synth.dense_f32(80, 0, n, kz)
    if bf16:
        X = oracle.bf16_to_f32(oracle.bf16_rne(X))
    Xd = torch.from_numpy(np.ascontiguousarray(X[bt.ref["gmap_r"]])).to(DEV)
    Xd = Xd.bfloat16() if bf16 else Xd
    y, my = oracle.spmm(bt.cols, bt.rows, 0, 0, bt.ref["lmap_c"], bt.ref["C"], bt.vals, X, 0, kz)
    Y1 = spc.spmm(bt.plan, bt.v, Xd, 1, kz)
    assert_within_mag(_np(Y1), y, my, what="transposed slices")
    vt = spc.permute_values(bt.plan, spc.SLOT_TO_COLUMN, bt.v)
    assert torch.equal(spc.spmm(bt.plan, vt, Xd, 2, kz), Y1)
