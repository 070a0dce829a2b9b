"""The small-step kernel's forms that the circuits of test_small_steps do not
hold, and a check that the two files together hold every form of the dispatch
(rows and columns per thread or block, one or eight wave sums, rows shared by a
whole block and read with scalar loads or not)."""
import numpy as np
import pytest

from paper_2211_17028_amd import tn
from tests.schedule_sim import Sim
from tests.test_small_steps import CASES, _circuit, _groups

# (fp64, split, log2 rows, log2 columns, scalar rows)
FORMS = {(0, 0, 0, 0, 0), (0, 0, 1, 0, 0), (0, 0, 2, 0, 0), (0, 0, 3, 0, 0), (0, 0, 0, 1, 0), (0, 0, 1, 1, 0),
         (0, 0, 2, 1, 0), (0, 0, 0, 1, 1), (0, 0, 1, 1, 1), (0, 0, 2, 1, 1), (0, 0, 0, 2, 1), (0, 0, 1, 2, 1),
         (0, 0, 2, 2, 1),
         (1, 0, 0, 0, 0), (1, 0, 1, 0, 0), (1, 0, 2, 0, 0), (1, 0, 3, 0, 0), (1, 0, 1, 0, 1), (1, 0, 2, 0, 1),
         (1, 0, 3, 0, 1),
         (0, 1, 0, 0, 0), (0, 1, 0, 1, 0), (0, 1, 1, 0, 0), (0, 1, 1, 1, 0), (0, 1, 1, 2, 0), (0, 1, 2, 1, 0),
         (0, 1, 2, 2, 0), (1, 1, 0, 0, 0), (1, 1, 0, 1, 0), (1, 1, 1, 0, 0), (1, 1, 1, 1, 0),
         (0, 2, 0, 0, 0), (1, 2, 0, 0, 0)}

# circuit, whether its exact value (doubled network) is what is computed, a form it holds
MORE = [(("chain", 120, 23, 12, 5), False, (0, 1, 1, 0, 0)), (("grid", 578, 24, 12, 5), False, (0, 0, 1, 2, 1)),
        (("grid", 202, 16, 12, 5), False, (1, 0, 3, 0, 1)), (("grid", 66, 12, 18, 4), True, (1, 0, 1, 0, 0)),
        (("grid", 972, 16, 11, 5), True, (1, 0, 3, 0, 0))]


def _schedule(case, doubled):
    circ = _circuit(*case)
    plan = tn.tn_plan_build_doubled(circ, path_trials=64) if doubled else tn.tn_plan_build(circ, 2, path_trials=64)
    terms = tn.tn_terms_enumerate(plan, 0 if doubled else 2)
    desc, cb = tn.tn_exec_describe_only([plan], [terms])
    return plan, terms, desc, cb


def _forms(desc):
    out = set()
    for j in (j for L in _groups(desc) for j in L["jobs"]):
        rl, cl = j["rpt_log"], j["cpt_log"]
        scalar = j["split"] == 0 and (cl > 0 or (j["fp64"] and rl > 0)) and j["n_log"] - cl >= 8
        out.add((j["fp64"], j["split"], rl, cl, int(scalar)))
    return out


def test_the_circuits_hold_every_form():
    held = set()
    for case, doubled in [(c, False) for c, _ in CASES] + [(c, d) for c, d, _ in MORE]:
        held |= _forms(_schedule(case, doubled)[2])
    assert held == FORMS


@pytest.mark.gpu
@pytest.mark.parametrize("case,doubled,form", MORE)
def test_form_matches_the_host_replay(case, doubled, form):
    print("small-step form", case, doubled, form, flush=True)
    plan, terms, desc, cb = _schedule(case, doubled)
    assert form in _forms(desc)
    _, w = terms.get()
    sim = Sim(desc, cb)
    sim.run([[i for i in range(terms.n) if w[i] != 0.0]])
    x_ref, a_ref = sim.outputs()
    ex = tn.tn_exec_prepare([plan], [terms])
    ex.run()
    x, a = ex.values()
    # FP32 sums in another order than numpy's, over up to 14 levels: errors of a
    # few 2^-24 per level against the amplitudes' norm; the dominant term in FP64
    # (an exact value: sums down to 2^-16 of the norms they are formed from)
    assert np.linalg.norm(a - a_ref) <= 1e-5 * np.linalg.norm(a_ref)
    assert abs(x[0] - x_ref[0]) <= (1e-9 if doubled else 1e-12) * abs(x_ref[0])
    ex.run()
    x2, a2 = ex.values()
    assert np.array_equal(x, x2) and np.array_equal(a, a2)
