"""Device memory of SPARSE circuits: whichever allocation of the first
evaluation fails, the next evaluation starts anew and is right."""
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
