"""The small-step launches: every shape of the dispatch (outputs per thread,
per block, per wave; FP32 and FP64; rows shared by a block or not) against the
host replay of the same schedule, and the rule that joins consecutive small
levels into one launch."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is the one the library binds to)

import workloads.circuits as WC
from paper_2211_17028_amd import tn
from tests.schedule_sim import Sim

# (kind, seed, qubits, layers, noises): circuits whose schedules hold the wanted
# (fp64, split, rpt_log, cpt_log) small steps
CASES = [
    (("chain", 319, 24, 12, 7), {(0, 0, 0, 2), (0, 1, 0, 1), (1, 1, 0, 1)}),
    (("chain", 481, 22, 12, 7), {(0, 0, 2, 1)}),
    (("chain", 406, 16, 11, 7), {(0, 0, 1, 1), (1, 1, 0, 1)}),
    (("chain", 406, 22, 12, 7), {(0, 1, 1, 2), (0, 2, 0, 0), (1, 2, 0, 0)}),
    (("chain", 905, 22, 10, 8), {(1, 1, 1, 0)}),
    (("grid", 5, 24, 7, 8), {(0, 0, 2, 1)}),
    (("grid", 992, 24, 9, 8), {(0, 0, 3, 0)}),
    (("grid", 955, 16, 11, 8), {(0, 0, 3, 0)}),
    (("grid", 100, 12, 11, 6), {(0, 0, 2, 0)}),
    (("grid", 604, 12, 8, 7), {(0, 1, 2, 2)}),
    (("grid", 284, 16, 11, 7), {(1, 1, 1, 1)}),
    (("grid", 655, 16, 12, 4), {(1, 0, 2, 0)}),
    (("qaoa", 274, 18, 2, 8), {(0, 0, 2, 2)}),
    (("qaoa", 879, 20, 2, 8), {(0, 0, 1, 0), (0, 0, 2, 0)}),
    (("qaoa", 885, 18, 2, 5), {(0, 1, 2, 1)}),
    (("qaoa", 396, 24, 2, 8), {(1, 0, 2, 0)}),
]


def _circuit(kind, seed, n, layers, noises):
    rng = np.random.default_rng(seed)
    if kind == "chain":
        gates = WC.chain_layers(n, layers, rng)
    elif kind == "grid":
        gates = WC.grid_layers(n // 4, 4, layers, "ABCD", rng)
    else:
        gates = WC.qaoa_3regular(n, layers, seed, rng)
    kraus = [WC.kraus_ad_pd(*rng.uniform(1e-3, 1e-2, 2)) for _ in range(noises)]
    return WC.Circuit(n, WC.place_noises(gates, kraus, rng), WC.zero_product(n), "circuit_output",
                      WC.zero_product(n), level=2)


def _schedule(case):
    circ = _circuit(*case)
    plan = tn.tn_plan_build(circ, 2, path_trials=64)
    terms = tn.tn_terms_enumerate(plan, 2)
    desc, cb = tn.tn_exec_describe_only([plan], [terms])
    return plan, terms, desc, cb


def _groups(desc):
    return [L for L in desc["launches"] if L["kind"] == 5]


@pytest.mark.gpu
@pytest.mark.parametrize("case,wanted", CASES, ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else "")
def test_every_shape_matches_the_host_replay(case, wanted):
    print("small steps", case, flush=True)
    plan, terms, desc, cb = _schedule(case)
    shapes = {(j["fp64"], j["split"], j["rpt_log"], j["cpt_log"]) for L in _groups(desc) for j in L["jobs"]}
    assert wanted <= shapes, shapes
    _, w = terms.get()
    sim = Sim(desc, cb)
    sim.run([[i for i in range(terms.n) if w[i] != 0.0]])
    x_ref, a_ref = sim.outputs()
    ex = tn.tn_exec_prepare([plan], [terms])
    ex.run()
    x, a = ex.values()
    # FP32 sums in another order than numpy's, over up to 14 levels: errors of a
    # few 2^-24 per level against the amplitudes' norm; the dominant term in FP64
    assert np.linalg.norm(a - a_ref) <= 1e-5 * np.linalg.norm(a_ref)
    assert abs(x[0] - x_ref[0]) <= 1e-12 * x_ref[0]
    ex.run()
    x2, a2 = ex.values()
    assert np.array_equal(x, x2) and np.array_equal(a, a2)


@pytest.mark.parametrize("case", [c for c, _ in CASES[::3]] + [("chain", 3, 8, 10, 4), ("grid", 7, 64, 6, 12),
                                                               ("chain", 11, 49, 13, 11)])
def test_joined_levels_are_independent_parts(case):
    """A chain launch has no order between its parts: none may touch memory that
    another one writes.  Within a part every level's blocks come before the next
    launch's, and the parts hold each block of the joined launches once."""
    _, _, desc, _ = _schedule(case)
    launches = desc["launches"]
    members = {}
    for i, L in enumerate(launches):
        if L["kind"] == 5 and L["chain"] >= 0:
            members.setdefault(L["chain"], []).append(i)
    assert sorted(members) == list(range(len(desc["chains"])))
    for ci, parts in enumerate(desc["chains"]):
        assert len(members[ci]) >= 2 and members[ci] == list(range(members[ci][0], members[ci][-1] + 1))
        blocks = [tuple(b) for p in parts for lv in p for b in lv]
        want = [(i, q, b) for i in members[ci] for q, j in enumerate(launches[i]["jobs"]) for b in range(j["blocks"])]
        assert sorted(blocks) == sorted(want)
        reads, writes = [], []
        for p in parts:
            assert [len({b[0] for b in lv}) for lv in p] == [1] * len(p)      # a level of a part: one launch
            assert all(p[k][0][0] < p[k + 1][0][0] for k in range(len(p) - 1))
            jobs = [launches[i]["jobs"][q] for i, q in sorted({(b[0], b[1]) for lv in p for b in lv})]
            span = lambda r, n: (r[0], r[1], r[1] + n)                        # noqa: E731
            writes.append([span(j["c"], j["len"][2]) for j in jobs])
            reads.append([span(j[o], j["len"][k]) for j in jobs for k, o in enumerate("ab")])
            assert all(j["rpt_log"] == j["cpt_log"] == 0 for j in jobs)
        cut = lambda s, t: s[0] == t[0] and s[1] < t[2] and t[1] < s[2]       # noqa: E731
        for x in range(len(parts)):
            for y in range(len(parts)):
                if x != y:
                    assert not any(cut(s, t) for s in writes[x] for t in writes[y] + reads[y])


@pytest.mark.parametrize("max_ksplit", [0, 1, 4])
def test_long_sums_follow_the_callers_split_limit(max_ksplit):
    """8 x 8 FP64 outputs over 2^18 terms: a split tile job, or the small-step
    kernel where the caller limits the split."""
    rng = np.random.default_rng(2)
    gates = WC.grid_layers(4, 4, 18, "ABCD", rng)
    kraus = [WC.kraus_ad_pd(*rng.uniform(1e-3, 1e-2, 2)) for _ in range(4)]
    circ = WC.Circuit(16, WC.place_noises(gates, kraus, rng), WC.zero_product(16), "circuit_output",
                      WC.zero_product(16), level=0)
    plan = tn.tn_plan_build_doubled(circ, path_trials=256)
    desc, _ = tn.tn_exec_describe_only([plan], [tn.tn_terms_enumerate(plan, 0)], tn.exec_opts(max_ksplit=max_ksplit))
    tiled = [(j["m_log"], j["n_log"], j["k_log"]) for L in desc["launches"] if L.get("kernel") == "k_tile64_group"
             for j in L["jobs"]]
    small = [(j["m_log"], j["n_log"], j["k_log"]) for L in _groups(desc) for j in L["jobs"]]
    assert ((3, 3, 18) in tiled) == (max_ksplit == 0) and ((3, 3, 18) in small) == (max_ksplit != 0)
