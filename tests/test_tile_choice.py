"""The tile shape that long sums of few rows and columns take."""
import workloads as W
from paper_2211_17028_amd import tn


def test_short_slices_over_long_sums_take_short_tiles():
    """36-qubit QAOA: 8208 slices of 8 x 16 outputs over 1024 terms run on 32 x 16
    tiles (four slices each, no padding columns), not on half-empty 128 x 32 ones
    (376 us against 261)."""
    circ = W.config(3)
    plan = tn.tn_plan_build(circ, 2)
    desc, _ = tn.tn_exec_describe_only([plan], [tn.tn_terms_enumerate(plan, 2)])
    tiles = [(L["bm"], L["bn"]) for L in desc["launches"] if L.get("kernel", "").startswith("k_mfma_group")
             for j in L["jobs"] if (j["m_log"], j["n_log"], j["k_log"]) == (3, 4, 10) and j["ns"] == 8208]
    assert tiles == [(32, 16)]

