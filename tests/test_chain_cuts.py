"""Where lists of small levels are cut into chain launches: the cut with the least
modelled time, found here by trying every cut."""
import itertools

import pytest

from paper_2211_17028_amd import tn
from tests.test_small_steps import _circuit

LAUNCH, ROUND, BATCH, BLOCKS, LEVELS = 3.5, 2.5, 0.6, 24, 24


def _round(L):
    batches = 1.0
    for j in L["jobs"]:
        k = 2.0 ** j["k_log"] / {0: 1, 1: 256, 2: 4}[j["split"]]
        batches = max(batches, k / ((8 if j["fp64"] else 16) if j["split"] == 1 else (4 if j["fp64"] else 8)))
    return ROUND + BATCH * batches


def _time(run):
    """Modelled time of consecutive launches as one."""
    if len(run) == 1:
        return LAUNCH + _round(run[0])
    jobs = [(lv, j) for lv, L in enumerate(run) for j in L["jobs"]]
    span = lambda j, o: (j[o][0], j[o][1], j[o][1] + j["len"]["abc".index(o)])           # noqa: E731
    cut = lambda s, t: s[0] == t[0] and s[1] < t[2] and t[1] < s[2]                       # noqa: E731
    part = list(range(len(jobs)))
    for x, y in itertools.combinations(range(len(jobs)), 2):
        (lx, p), (ly, q) = jobs[x], jobs[y]
        if lx != ly and (any(cut(span(p, "c"), span(q, o)) for o in "abc") or
                         any(cut(span(q, "c"), span(p, o)) for o in "ab")):
            a, b = part[x], part[y]
            part = [a if v == b else v for v in part]
    longest = 0.0
    for r in set(part):
        t = 0.0
        for lv, L in enumerate(run):
            n = sum(j["blocks"] for i, (l, j) in enumerate(jobs) if l == lv and part[i] == r)
            if n > BLOCKS:
                return 1e300
            t += _round(L) * -(-n // 4)
        longest = max(longest, t)
    return LAUNCH + longest


@pytest.mark.parametrize("case", [("chain", 3, 8, 10, 4), ("grid", 7, 64, 6, 12), ("grid", 5, 16, 9, 5),
                                  ("chain", 21, 20, 11, 3), ("qaoa", 9, 12, 1, 6), ("chain", 2, 7, 14, 9)])
def test_lists_are_cut_where_their_time_is_least(case):
    circ = _circuit(*case)
    plan = tn.tn_plan_build(circ, 2, path_trials=64)
    desc, _ = tn.tn_exec_describe_only([plan], [tn.tn_terms_enumerate(plan, 2)])
    for phase in ("const", "batch64", "batch"):
        runs, last = [], None
        for i, L in enumerate(L for L in desc["launches"] if L["phase"] == phase):
            if L["kind"] == 5 and all(j["rpt_log"] == j["cpt_log"] == 0 and j["blocks"] <= BLOCKS for j in L["jobs"]):
                if last != i - 1:
                    runs.append([])
                runs[-1].append(L)
                last = i
            elif L["kind"] == 5:
                assert L["chain"] == -1
        for run in runs:
            best = [0.0] + [1e300] * len(run)
            for i in range(len(run)):
                for e in range(i + 1, min(len(run), i + LEVELS) + 1):
                    best[e] = min(best[e], best[i] + _time(run[i:e]))
            groups = [list(g) for _, g in itertools.groupby(enumerate(run), key=lambda q: (q[1]["chain"], q[1]["chain"] < 0 and q[0]))]
            taken = sum(_time([L for _, L in g]) for g in groups)
            assert taken == pytest.approx(best[-1], rel=1e-12)
