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



def packed_tiles(cfg):
    circ = W.config(cfg)
    plans = [tn.tn_plan_build(circ, 2) for _ in range(2)]
    desc, _ = tn.tn_exec_describe_only(plans, [tn.tn_terms_enumerate(p, 2) for p in plans])
    return [(L["level"], (L["bm"], L["bn"]), {(j["m_log"], j["n_log"], j["k_log"]) for j in L["jobs"]})
            for L in desc["launches"] if L.get("kernel", "").startswith("k_mfma_group")]


def test_heavy_packed_levels_take_wide_tiles():
    """Two 36-qubit QAOA circuits: 396 slices of 128 x 512 outputs each fill 128 x 64
    tiles, which read the rows half as often as 128 x 32 ones; the same level's slices
    of 16 columns stay on 128 x 32."""
    tile = {shape: bmn for _, bmn, jobs in packed_tiles(3) for shape in jobs}
    assert tile[(7, 9, 4)] == (128, 64)
    assert tile[(14, 4, 3)] == (128, 32)


def test_light_packed_levels_take_one_launch():
    """Two 25-qubit grids: no level's work pays for a second tile shape."""
    levels = [level for level, _, jobs in packed_tiles(2) if any(k < 9 and m + n + k >= 18 for m, n, k in jobs)]
    assert levels and len(levels) == len(set(levels))
