"""The launches of one estimate as a schedule's description counts them."""
import pytest

import workloads as W
from paper_2211_17028_amd import tn


@pytest.mark.parametrize("circ,level,launches", [(W.config(1, level=2), 2, 2), (W.config(2), 2, None),
                                                 (W.config(5), 3, None)], ids=["chain8", "grid25", "grid225"])
def test_joined_levels_count_once(circ, level, launches):
    """8-qubit chain: its three levels in one launch and the tail in one."""
    plan = tn.tn_plan_build(circ, level)
    terms = tn.tn_terms_enumerate(plan, level)
    desc, _ = tn.tn_exec_describe_only([plan], [terms])
    main = [L for L in desc["launches"] if L["phase"] in ("batch", "batch64")]
    chains = {L["chain"] for L in main if L["kind"] == 5 and L["chain"] >= 0}
    alone = sum(1 for L in main if not (L["kind"] == 5 and L["chain"] >= 0))
    assert desc["estimate_launches"] == alone + len(chains) + (1 if terms.n <= 2048 else 2)
    assert launches is None or desc["estimate_launches"] == launches
    # timed launch by launch: no level is joined
    timed, _ = tn.tn_exec_describe_only([plan], [terms], tn.exec_opts(time_kernels=True))
    assert timed["estimate_launches"] == len(main) + (1 if terms.n <= 2048 else 2)
