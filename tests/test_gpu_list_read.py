"""Reading a list after its evaluation takes no device memory and may be
repeated, before and after further evaluations."""
import numpy as np
import pytest

from paper_2502_10685_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,graph", [(33, 0), (34, 1), (48, 0), (64, 1)])
def test_terms_without_memory(n, graph, dtype):
    import torch
    from paper_2502_10685_amd import _lib as L
    from paper_2502_10685_amd import api
    assert torch.cuda.is_available(), "GPU tests need a visible HIP device"
    print(f"list read n={n} graph={graph} {dtype}", flush=True)
    w = W.random_circuit(np.random.default_rng(n), n, 260, W.obs_tfim(n))
    c = api.Circuit.from_workload(w, engine="sparse", dtype=dtype, max_terms=1 << 18)
    c.set_truncation(1e-3, 64)
    c.set_option(L.PP_OPT_USE_GRAPH, graph)
    ev = float(c.evaluate().item())
    want = None
    api.set_allocator(lambda nbytes: None, lambda ptr: None)
    try:
        for _ in range(3):
            for _ in range(2):
                got = c.terms(capacity=1 << 18)
                keys = [(int(b), int(a)) for a, b in zip(got[0], got[1])]
                assert len(keys) > 64 and keys == sorted(set(keys))
                assert want is None or all(a.tobytes() == b.tobytes() for a, b in zip(want, got))
                want = got
            assert float(c.evaluate().item()) == ev
    finally:
        api.set_allocator()
    c.close()
