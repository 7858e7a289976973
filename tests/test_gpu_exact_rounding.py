"""The exact sum of a list is rounded once: where workgroups' shares cancel, the
readout is still the correctly rounded sum, whichever workgroup held what."""
import math

import numpy as np
import pytest

from paper_2502_10685_amd import workloads as W

pytestmark = pytest.mark.gpu

TIE = [2.0 ** -60, 2.0 ** -113, 2.0 ** -140]  # just above the middle of two doubles


def _spread(values, at, count=900):
    v = np.zeros(count)
    v[at] = values
    return v


def _cases():
    rng = np.random.default_rng(3)
    big = rng.standard_normal(450) * 10.0 ** rng.uniform(-30, 30, 450)
    return {
        "tie_up": _spread([1.0, -1.0, *TIE], [0, 256, 10, 300, 600]),
        "tie_down": _spread([1.0, -1.0, TIE[0], TIE[1], -TIE[2]], [0, 256, 10, 300, 600]),
        "negative": -_spread([1.0, -1.0, *TIE], [0, 256, 10, 300, 600]),
        "to_even": _spread([-1.0, 1.0, 1.0 + 2.0 ** -52, 2.0 ** -53], [0, 700, 300, 600]),
        "cancels_but_one": np.concatenate([big, [5e-324], -rng.permutation(big)]),
        "cancels": np.concatenate([big, -rng.permutation(big)]),
        "subnormal": _spread([2.0 ** -1022, -5e-324, -(2.0 ** -1030)], [0, 300, 600]),
        "largest": _spread([1.7976931348623157e308, 2.0 ** 970, -(2.0 ** 960)], [0, 300, 600]),
        "beyond": _spread([1.7976931348623157e308, 1.7976931348623157e308], [0, 600]),
        "back": _spread([1.7976931348623157e308, 1.7976931348623157e308, -1.7976931348623157e308], [0, 600, 300]),
    }


@pytest.mark.parametrize("frame", [0, 1])
@pytest.mark.parametrize("kind", list(_cases()))
def test_readout_is_rounded_once(kind, frame):
    import torch
    from paper_2502_10685_amd import _lib as L
    from paper_2502_10685_amd import api
    assert torch.cuda.is_available(), "GPU tests need a visible HIP device"
    v = _cases()[kind]
    arr = tuple(np.array(a, dtype=t) for a, t in zip(([W.CX], [11], [10], [-1]), (np.uint8, np.int32, np.int32, np.int32)))
    wc = W.make_circuit(12, arr, 0, W.observable([(0, k + 1, float(t)) for k, t in enumerate(v)]), [])
    c = api.Circuit.from_workload(wc, engine="sparse", max_terms=1 << 12)
    c.set_option(L.PP_OPT_SPARSE_FRAME, frame)
    try:
        want = math.fsum(sorted(v.tolist(), key=abs))
    except OverflowError:
        want = math.inf
    if kind == "back":
        want = 1.7976931348623157e308
    for _ in range(2):
        assert float(c.evaluate().item()) == want
    c.close()
