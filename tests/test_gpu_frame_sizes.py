"""The Clifford-frame engine at the sizes where its passes change: one string
per thread up to the grid's threads, several beyond, and capacities whose
index has fewer than four slots.  Z...Z under an RX on every qubit gives 2^n
strings and <O> = prod cos.

Tolerance: n roundings of a product, 4 units in the last place each."""
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


def _product(n, theta):
    arr = [np.array(a, dtype=t) for a, t in zip(([W.RX] * n, list(range(n)), [-1] * n, list(range(n))),
                                                (np.uint8, np.int32, np.int32, np.int32))]
    return W.make_circuit(n, tuple(arr), n, W.obs_z(n, range(n)), theta)


@pytest.mark.parametrize("n,cap,dtype", [(1, 2, "f64"), (8, 1 << 8, "f64"), (19, 1 << 19, "f64"), (21, 1 << 21, "f64"),
                                         (21, 1 << 24, "f32"), (12, 1 << 20, "f32")])
def test_product_strings(api, n, cap, dtype):
    print(f"frame product n={n} cap={cap} {dtype}", flush=True)
    theta = np.random.default_rng(n).uniform(0.1, 0.6, size=n)
    c = api.Circuit.from_workload(_product(n, theta), engine="sparse", dtype=dtype, max_terms=cap)
    tol = 8 * n * (2.0 ** -53 if dtype == "f64" else 2.0 ** -24)
    for _ in range(2):
        assert abs(float(c.evaluate().item()) - np.prod(np.cos(theta))) <= tol
        assert c.stats()["final_terms"] == 1 << n and c.stats()["term_updates"] == (1 << n) - 1
    x, z, v = c.terms(capacity=1 << n)
    ref = np.ones(1)
    for t in theta:  # qubit q is bit q of x
        ref = np.concatenate([ref * math.cos(t), ref * math.sin(t)])
    assert np.array_equal(x, np.arange(1 << n, dtype=np.uint64)) and np.all(z == (1 << n) - 1)
    assert float(np.max(np.abs(v - ref))) <= tol
    c.close()


@pytest.mark.parametrize("n,cap", [(1, 1), (9, (1 << 9) - 1), (20, (1 << 20) - 1)])
def test_one_string_too_many(api, n, cap):
    c = api.Circuit.from_workload(_product(n, np.full(n, 0.3)), engine="sparse", max_terms=cap)
    assert math.isnan(float(c.evaluate().item())) and c.stats()["overflow"]
    c.close()
