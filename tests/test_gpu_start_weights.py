"""Start weights written in parallel (distinct strings) or in input order
(repeats), and long recipes spread over waves, against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_2502_10685_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2502_10685_amd import api as a
    return a


# one string, just above one block's threads, every string; n = 9 is tiled
@pytest.mark.parametrize("n,nterms,repeat", [(3, 1, False), (4, 255, False), (5, 257, False), (5, 257, True),
                                             (9, 1, True), (9, 1025, False), (9, 1025, True)])
def test_observable_terms(api, n, nterms, repeat):
    rng = np.random.default_rng([n, nterms, repeat])
    wc = W.random_circuit(rng, n, 60)
    slots = rng.choice(4 ** n, size=nterms, replace=False).astype(np.uint64)
    x, z = slots & np.uint64(2 ** n - 1), slots >> np.uint64(n)
    c = rng.uniform(-1, 1, size=nterms)
    if repeat:
        x, z, c = np.tile(x, 2), np.tile(z, 2), np.concatenate([c, rng.uniform(-1, 1, size=nterms)])
    wc = W.make_circuit(n, (wc.op, wc.q0, wc.q1, wc.param), wc.n_params, (x, z, c), wc.theta)
    got = api.Circuit.from_workload(wc).evaluate().item()
    # 1e-12 per unit of the observable's norm, the FP64 bar of one string
    assert abs(got - oracle.expval_sv(wc)) <= 1e-12 * max(1.0, np.abs(c).sum())


# recipes at the edges of the one-lane rule (8 gates) and of a 64-gate chunk
@pytest.mark.parametrize("repeats", [2, 3, 21, 22, 43])
def test_long_recipes(api, repeats):
    wc = W.chain_zxz_circuit(seed=repeats, n=3, layers=5, repeats=repeats)
    got = api.Circuit.from_workload(wc).evaluate().item()
    assert abs(got - oracle.expval_sv(wc)) <= 1e-12
