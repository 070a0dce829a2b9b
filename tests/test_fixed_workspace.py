"""Workspaces below the size that the model's schedule asks for.  The sizes here
are those of schedules whose split sums take less scratch: they are served by
one schedule, not refused and not cut into term ranges."""
import ctypes as C

import numpy as np
import pytest

import workloads.circuits as WC
from paper_2211_17028_amd import tn

# (kind, seed, qubits, layers, noises), bytes of an estimate, of all terms' amplitudes
CASES = [(("chain", 47, 38, 12, 8), 64069888, 36130048), (("grid", 67, 20, 9, 11), 26143744, 23196672),
         (("chain", 143, 58, 14, 6), 35050240, 18066944), (("grid", 21, 16, 10, 10), 279023360, 255518976)]


def _plan(kind, seed, n, layers, noises):
    rng = np.random.default_rng(seed)
    gates = WC.chain_layers(n, layers, rng) if kind == "chain" else WC.grid_layers(n // 4, 4, layers, "ABCD", rng)
    kraus = [WC.kraus_ad_pd(*rng.uniform(1e-3, 1e-2, 2)) for _ in range(noises)]
    circ = WC.Circuit(n, WC.place_noises(gates, kraus, rng), WC.zero_product(n), "circuit_output",
                      WC.zero_product(n), level=2)
    plan = tn.tn_plan_build(circ, 2, path_trials=64)
    return plan, tn.tn_terms_enumerate(plan, 2)


@pytest.mark.parametrize("case,full,batch", CASES)
def test_the_size_check_takes_the_smaller_schedule(case, full, batch):
    """Without a device: past the size check a call ends at its first device call.
    (The pointers are not device memory: not run where there is a device.)"""
    import torch
    if torch.cuda.is_available():
        pytest.skip("the pointers here are not device memory")
    plan, terms = _plan(*case)
    assert tn.tn_plan_workspace([plan], [terms])[1] > full
    L, P, T = tn.lib(), tn._handles([plan]), tn._handles([terms])
    fake, amp, h, need = C.c_void_p(4096), C.c_void_p(8192), C.c_void_p(), C.c_size_t()
    o = tn.exec_opts()
    assert L.tn_exec_prepare(1, P, T, C.byref(o), fake, full, None, C.byref(need), C.byref(h)) == tn.TN_EHIP
    assert need.value <= full
    assert L.tn_contract_batch(1, P, T, 0, terms.n, amp, fake, batch, None) == tn.TN_EHIP
    assert L.tn_contract_batch(1, P, T, 0, terms.n, amp, fake, batch // 2, None) == tn.TN_ENOMEM
    assert L.tn_exec_prepare(1, P, T, C.byref(o), fake, full // 2, None, C.byref(need), C.byref(h)) == tn.TN_ENOMEM


@pytest.mark.gpu
@pytest.mark.parametrize("case,full,batch", CASES)
def test_values_of_the_smaller_schedule(case, full, batch):
    import torch
    print("fixed workspace", case, flush=True)
    plan, terms = _plan(*case)
    ex = tn.tn_exec_prepare([plan], [terms])
    want = ex.run()[0]
    L, P, T = tn.lib(), tn._handles([plan]), tn._handles([terms])
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    ptr = lambda t: C.c_void_p(t.data_ptr())                                   # noqa: E731
    o, h, need = tn.exec_opts(), C.c_void_p(), C.c_size_t()
    tn._check(L.tn_exec_prepare(1, P, T, C.byref(o), ptr(ws), full, None, C.byref(need), C.byref(h)))
    assert need.value <= full
    small = tn.Exec(h, [plan], [terms], ws, need.value)
    got = small.run()[0]
    # FP32 sums in another order over up to 15 levels: a few 2^-24 per level; the
    # dominant term in FP64
    for u in range(3):
        assert abs(got["A"][u] - want["A"][u]) <= 1e-6 * abs(want["A"][u])
    assert abs(got["T"][0] - want["T"][0]) <= 1e-12 * abs(want["T"][0])
    del small
    res = (tn.tn_result * 1)()
    tn._check(L.tn_estimate(1, P, T, ptr(ws), full, None, res))
    assert res[0].A[2] == got["A"][2]               # one schedule, the same one
    amp = torch.empty(2 * terms.n, dtype=torch.float32, device="cuda")
    tn._check(L.tn_contract_batch(1, P, T, 0, terms.n, ptr(amp), ptr(ws), batch, None))
    torch.cuda.synchronize()
    a = amp.cpu().numpy().view(np.complex64)
    a_ref = ex.values()[1]
    assert np.linalg.norm(a - a_ref) <= 1e-5 * np.linalg.norm(a_ref)
    tn.tn_release_cached()


@pytest.mark.gpu
def test_noalloc_is_the_estimate_of_a_64_MiB_workspace():
    """The model's schedule of this chain needs 72 MB, the smaller one 64 MB."""
    import torch
    print("noalloc at its limit", flush=True)
    plan, terms = _plan(*CASES[0][0])
    assert tn.tn_plan_workspace([plan], [terms])[1] > 64 << 20
    got = tn.tn_estimate_noalloc([plan], [terms])[0]
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    res = (tn.tn_result * 1)()
    tn._check(tn.lib().tn_estimate(1, tn._handles([plan]), tn._handles([terms]), C.c_void_p(ws.data_ptr()), 64 << 20,
                                   None, res))
    assert list(got["A"]) == list(res[0].A)[:3]
    tn.tn_release_cached()
