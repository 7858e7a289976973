"""A gradient's schedule follows the tile size asked for, whatever was evaluated
before: the option set after a first gradient gives the bits of a circuit that
had it from the start."""
import numpy as np
import pytest

from paper_2502_10685_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_tile_option_after_a_gradient():
    import torch
    from paper_2502_10685_amd import _lib as L
    from paper_2502_10685_amd import api
    assert torch.cuda.is_available(), "GPU tests need a visible HIP device"
    w = W.random_circuit(np.random.default_rng(31), 10, 900, W.obs_tfim(10))

    def bits(c):
        ev, g = c.gradient()
        return float(ev.item()), g.cpu().numpy().tobytes()

    fresh = {}
    for k in (6, 7):
        c = api.Circuit.from_workload(w, tile_qubits=k)
        fresh[k] = bits(c)
        c.close()
    assert fresh[6] != fresh[7]
    c = api.Circuit.from_workload(w)
    c.evaluate()
    bits(c)
    for k in (7, 6, 7):
        c.set_option(L.PP_OPT_TILE_QUBITS, k)
        assert bits(c) == fresh[k]
    c.close()
