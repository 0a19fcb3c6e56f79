"""The committed networks on timings in which the default shape (variant -1) is
the one the library takes now, with the run family where it applies: the
autotuner's records of the 128 held-out blocks.  On these the networks trained
before the run family chose shapes 4% (SpMM) and 8% (fused) slower than the
default in the geometric mean."""
import os

import pytest

torch = pytest.importorskip("torch")
pytestmark = [
    pytest.mark.gpu,
    pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU"),
]
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("op", ["sddmm", "spmm", "sddmm_spmm"])
def test_no_choice_is_slower_than_the_present_default(op):
    from paper_2404_19638_amd import selector as S
    from paper_2404_19638_amd import synth
    sel = S.Selector.from_state(S.load_weights(os.path.join(
        ROOT, "paper_2404_19638_amd", "selector_weights.json")), "cuda:0")
    recs = S.load_records_npz(os.path.join(
        ROOT, "tests", "data", "selector_heldout_records_run_family.npz"))
    assert {r["block"] for r in recs} <= set(synth.selector_split(512, 384)[1])
    j = S.judge(sel, recs, op, S.best_fixed(recs, op))
    assert j["n"] == 1024
    assert j["regret_geomean"] <= j["default_regret_geomean"] + 1e-12, j
    assert j["gain_vs_fixed_geomean"] > 1.0, j
