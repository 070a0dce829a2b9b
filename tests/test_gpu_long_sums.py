"""FP64 inner products of few outputs over 2^17 terms and more: they run as tile
jobs split over many blocks although their slices fill only part of a tile.
Exact values of 16-qubit circuits that hold one, against the host replay of the
same schedule."""
import numpy as np
import pytest

import workloads.circuits as WC
from paper_2211_17028_amd import tn
from tests.schedule_sim import Sim

pytestmark = pytest.mark.gpu


# layers, seed, (row bits, column bits, inner bits) of the step
@pytest.mark.parametrize("layers,seed,shape", [(16, 0, (4, 4, 18)), (18, 0, (3, 4, 17)), (18, 2, (3, 3, 18)),
                                               (22, 4, (3, 4, 17))])
def test_long_sum_of_a_part_filled_tile(layers, seed, shape):
    import torch  # noqa: F401
    print("long sum", layers, seed, flush=True)
    rng = np.random.default_rng(seed)
    gates = WC.grid_layers(4, 4, layers, "ABCD", rng)
    kraus = [WC.kraus_ad_pd(*rng.uniform(1e-3, 1e-2, 2)) for _ in range(4)]
    circ = WC.Circuit(16, WC.place_noises(gates, kraus, rng), WC.zero_product(16), "circuit_output",
                      WC.zero_product(16), level=0)
    plan = tn.tn_plan_build_doubled(circ, path_trials=256)
    terms = tn.tn_terms_enumerate(plan, 0)
    desc, cb = tn.tn_exec_describe_only([plan], [terms])
    jobs = [j for L in desc["launches"] if L.get("kernel") == "k_tile64_group" for j in L["jobs"]]
    job, = [j for j in jobs if (j["m_log"], j["n_log"], j["k_log"]) == shape]
    assert job["ksplit"] > 16
    sim = Sim(desc, cb)
    sim.run([[0]])
    x_ref = sim.outputs()[0]
    ex = tn.tn_exec_prepare([plan], [terms])
    ex.run()
    # FP64 sums in another order over about 30 levels, the value down to 2^-16 of
    # the norms it is summed from: 30 x 2^-53 x 2^16 = 2e-10
    assert abs(ex.values()[0][0] - x_ref[0]) <= 1e-9 * abs(x_ref[0])
    first = ex.values()[0][0]
    ex.run()
    assert ex.values()[0][0] == first
