"""stats()["launches"] of tiled circuits: maps, steps and readout, and the two
launches that write the start weights only where the first passes do not."""
import numpy as np
import pytest

from paper_2502_10685_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8, 11])
def test_launches_of_tiled_circuits(n):
    import torch
    from paper_2502_10685_amd import _lib as L
    from paper_2502_10685_amd import api
    assert torch.cuda.is_available(), "GPU tests need a visible HIP device"
    rng = np.random.default_rng(n)
    many = W.observable([(0, k + 1, 1.0) for k in range(65)])  # more strings than a pass begins with
    for obs, extra in ((W.obs_tfim(n), 0), (many, 2)):
        w = W.random_circuit(rng, n, 300, obs)
        c = api.Circuit.from_workload(w)
        ev = float(c.evaluate().item())
        st = c.stats()
        assert st["launches"] == st["passes"] + 2 + extra
        k = st["tile_qubits"]
        old = L.tune_get(L.PP_TUNE_TILE_KERNEL, k)
        try:  # one workgroup per tile: it reads its start weights
            L.tune_set(L.PP_TUNE_TILE_KERNEL, k, 0)
            assert float(c.evaluate().item()) == ev
            assert c.stats()["launches"] == st["passes"] + 4
        finally:
            L.tune_set(L.PP_TUNE_TILE_KERNEL, k, old)
        c.close()
