"""The readout of the string lists is summed exactly: it is the correctly
rounded sum (to two units in the last place) of the weights of the I/Z strings
that pp_get_terms gives, whatever their sizes, signs and number, the same bits
on every call; the dropped weight is the same on every call."""
import math

import numpy as np
import pytest

from paper_2502_10685_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible HIP device"
    from paper_2502_10685_amd import api as A
    return A


def _z_terms(n, values):
    return W.observable([(0, k + 1, float(v)) for k, v in enumerate(values)])


@pytest.mark.parametrize("frame", [0, 1])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("kind", ["one", "tiny", "cancel", "range", "inf", "nan"])
def test_readout_is_the_exact_sum(api, frame, dtype, kind):
    from paper_2502_10685_amd import _lib as L
    rng = np.random.default_rng(5)
    top = 300 if dtype == "f64" else 30
    v = {"one": [0.1], "tiny": [5e-324, 1e-310] if dtype == "f64" else [1e-42, 1e-40],
         "cancel": [1.0, 1e16, -1e16, 2.0 ** -60, -1.0, 3e-17] * 50,
         "range": np.concatenate([s * 10.0 ** rng.uniform(-top, top / 2, size=300) for s in (1, -1)]),
         "inf": [1.0, math.inf, 2.0], "nan": [math.inf, -math.inf, 1.0]}[kind]
    n = 10
    # a CX, so that there is a pass
    arr = tuple(np.array(a, dtype=t) for a, t in zip(([W.CX], [8], [9], [-1]), (np.uint8, np.int32, np.int32, np.int32)))
    wc = W.make_circuit(n, arr, 0, _z_terms(n, v), [])
    c = api.Circuit.from_workload(wc, engine="sparse", dtype=dtype, max_terms=1 << 12)
    c.set_option(L.PP_OPT_SPARSE_FRAME, frame)
    ev = float(c.evaluate().item())
    x, _, w = c.terms(capacity=1 << 12)
    if kind == "nan":
        assert math.isnan(ev)
    elif kind == "inf":
        assert ev == math.inf
    else:
        exact = math.fsum(float(t) for a, t in zip(x, w) if a == 0)
        assert abs(ev - exact) <= 2 * math.ulp(exact)
    c.close()


def test_sums_are_the_same_on_every_call(api):
    wc = W.random_circuit(np.random.default_rng(22), 34, 260, W.obs_tfim(34))
    c = api.Circuit.from_workload(wc, engine="sparse", max_terms=1 << 20)
    c.set_truncation(1e-4, 12)
    first = None
    for _ in range(4):
        ev = float(c.evaluate().item())
        x, z, v = c.terms(capacity=1 << 20)
        got = (ev, c.truncation_dropped(), x.tobytes(), z.tobytes(), v.tobytes())
        assert first is None or got == first
        first = got
    exact = math.fsum(float(t) for a, t in zip(x, v) if a == 0)
    assert abs(first[0] - exact) <= 2 * math.ulp(exact)
    assert first[1] > 0.0
    c.close()
