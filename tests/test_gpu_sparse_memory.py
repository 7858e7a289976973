"""Device memory of SPARSE circuits: whichever allocation of the first
evaluation fails, the next evaluation starts anew and is right; the hash tables
of list passes are allocated for those alone, and a server counts them."""
import numpy as np
import pytest

import oracle
from paper_2502_10685_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible HIP device"
    from paper_2502_10685_amd import api as A
    return A


def _hooks(allowed):
    """torch's caching allocator, for `allowed` blocks."""
    import torch
    left = [allowed]

    def alloc(nbytes):
        left[0] -= 1
        return torch.cuda.caching_allocator_alloc(nbytes) if left[0] >= 0 else None

    return alloc, torch.cuda.caching_allocator_delete


@pytest.mark.parametrize("eps", [0.0, 1e-9])
def test_evaluation_after_any_failed_allocation(api, eps):
    from paper_2502_10685_amd._lib import PauliPropError, PP_ERR_NOMEM
    w = W.random_circuit(np.random.default_rng(8), 7, 120, W.obs_tfim(7))
    want = oracle.expval_sv(w)
    for allowed in range(60):
        print(f"sparse memory: eps={eps} {allowed} blocks", flush=True)
        api.set_allocator()
        c = api.Circuit.from_workload(w, engine="sparse", max_terms=1 << 14)
        c.set_truncation(min_abs_coeff=eps)
        alloc, free = _hooks(allowed)
        api.set_allocator(alloc, free)
        error = None
        try:
            c.evaluate()
        except PauliPropError as e:
            error = e
        finally:
            api.set_allocator()
        assert error is None or error.status == PP_ERR_NOMEM
        assert abs(float(c.evaluate().item()) - want) <= 1e-6
        c.close()
        if error is None:
            break
    assert 10 <= allowed < 59


def test_tables_only_for_list_passes(api):
    from paper_2502_10685_amd._lib import memory_in_use
    cap = 1 << 16
    tables = 3 * 4 << 18  # three of the power of two above 2 cap positions
    w = W.random_circuit(np.random.default_rng(9), 12, 100, W.obs_z(12, [0, 1]))
    c = api.Circuit.from_workload(w, engine="sparse", max_terms=cap)
    first = float(c.evaluate().item())  # exact: the Clifford frame
    frame = memory_in_use()[0]
    c.set_truncation(min_abs_coeff=1e-12)
    assert abs(float(c.evaluate().item()) - first) <= 1e-9
    assert abs(memory_in_use()[0] - frame - tables) <= 1 << 16  # and the schedules' own arrays
    c.set_truncation(min_abs_coeff=0.0)
    assert float(c.evaluate().item()) == first
    c.close()


def test_server_counts_the_tables(api):
    cap = 1 << 16
    arrays, tables = 64 * cap, 3 * 4 << 18
    ws = [W.random_circuit(np.random.default_rng(70 + i), 34, 300, W.obs_tfim(34)) for i in range(6)]

    def made(w):
        c = api.Circuit.from_workload(w, engine="sparse", max_terms=cap)
        c.set_truncation(1e-3, 10)
        return c

    solo = []
    for w in ws:
        c = made(w)
        solo.append(float(c.evaluate().item()))
        c.close()
    for budget, most in ((arrays, 1), (2 * (arrays + tables) - 1, 1), (2 * (arrays + tables), 2)):
        srv = api.Server(mem_budget_bytes=budget, max_active=16)
        circs = [made(w) for w in ws]
        tickets = [srv.submit(c) for c in circs]
        srv.drain()
        assert [srv.poll(t)[0] for t in tickets] == solo
        assert srv.counters()["max_in_flight"] <= most
        srv.close()
        for c in circs:
            c.close()
