"""Setting a tuned tile size back to what pp_tune_get gave restores the library's
own choice, which at n = 10 also looks at the circuit."""
import numpy as np
import pytest

from paper_2502_10685_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_default_tile_size_can_be_set_back():
    import torch
    from paper_2502_10685_amd import _lib as L
    from paper_2502_10685_amd import api
    assert torch.cuda.is_available(), "GPU tests need a visible HIP device"

    def chosen():
        out = []
        for m, track in ((900, False), (200, False), (900, True)):
            w = W.random_circuit(np.random.default_rng(m), 10, m, W.obs_z(10, [0]))
            c = api.Circuit.from_workload(w, track=track)
            c.evaluate()
            out.append(c.stats()["tile_qubits"])
            c.close()
        return out

    default = L.tune_get(L.PP_TUNE_TILE_QUBITS, 10)
    before = chosen()
    try:
        L.tune_set(L.PP_TUNE_TILE_QUBITS, 10, default)
        assert chosen() == before
        L.tune_set(L.PP_TUNE_TILE_QUBITS, 10, 5)
        assert chosen() == [5, 5, 5]
    finally:
        L.tune_set(L.PP_TUNE_TILE_QUBITS, 10, default)
    assert chosen() == before
