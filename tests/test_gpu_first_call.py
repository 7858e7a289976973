"""A first evaluation puts a DENSE schedule on the device as one block: beside it
only the circuit's weights (both ends' where it has two) and its two small
result buffers are allocated."""
import numpy as np
import pytest

import oracle
from paper_2502_10685_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,arrays", [(4, 0), (6, 0), (7, 0), (8, 2), (10, 2), (11, 1)])
def test_allocations_of_a_first_evaluation(n, arrays):
    import torch
    from paper_2502_10685_amd import api
    assert torch.cuda.is_available(), "GPU tests need a visible HIP device"
    print(f"first call n={n}", flush=True)
    w = W.random_circuit(np.random.default_rng(n), n, 400, W.obs_tfim(n))
    sizes = []

    def alloc(nbytes):
        sizes.append(nbytes)
        return torch.cuda.caching_allocator_alloc(nbytes)

    api.set_allocator()
    c = api.Circuit.from_workload(w)
    api.set_allocator(alloc, torch.cuda.caching_allocator_delete)
    try:
        ev = float(c.evaluate().item())
    finally:
        api.set_allocator()
    assert abs(ev - oracle.expval_sv(w)) <= 1e-12
    weights = [s for s in sizes if s == 8 * 4 ** n]
    assert len(weights) <= max(arrays, 1) and len(sizes) <= len(weights) + 3
    assert float(c.evaluate().item()) == ev
    c.close()
