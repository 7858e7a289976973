"""The adjoint sweep over composed runs: runs longer than a map may fold (255
gates), shared parameters, tiles of 1 to 6 digits, digit pairs without maps,
and sums flushed before the last segment, against the parameter-shift rule on
the oracle's state vector.

Tolerance: both derivatives are sums of 2-norm 1 vectors taken through m
rotations, 4 m 2^-53 each, and the observables here have at most n terms of
weight 1: 16 n m 2^-53, at least 1e-12."""
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


def _shift(wc, p):
    """Sum of the halved differences of the gates of parameter p."""
    g = 0.0
    for i in np.nonzero((wc.op >= 3) & (wc.param == p))[0]:
        param = wc.param.copy()
        param[i] = wc.n_params
        for s in (1, -1):
            theta = np.append(wc.theta, wc.theta[p] + s * np.pi / 2)
            v = W.Circuit(wc.n, wc.op, wc.q0, wc.q1, param, theta, wc.obs_x, wc.obs_z, wc.obs_c)
            g += s * 0.5 * oracle.expval_sv(v)
    return g


def _check(api, wc, every, params):
    print(f"adjoint n={wc.n} m={wc.m} every={every}", flush=True)
    c = api.Circuit.from_workload(wc)
    ev, g = c.gradient(every)
    tol = max(1e-12, 16 * wc.n * wc.m * 2.0 ** -53)
    assert abs(float(ev.item()) - oracle.expval_sv(wc)) <= tol
    g = g.cpu().numpy()
    for p in params:
        assert abs(g[p] - _shift(wc, p)) <= tol, (p, g[p])
    ev2, g2 = c.gradient(every)
    assert float(ev2.item()) == float(ev.item()) and np.array_equal(g2.cpu().numpy(), g)
    c.close()


@pytest.mark.parametrize("n", [1, 2, 6, 7])
def test_long_runs_and_shared_parameters(api, n):
    rng = np.random.default_rng(n)
    m = 600
    op = rng.integers(0, 6, size=m).astype(np.uint8)
    op[op == W.CX] = W.RY  # runs of up to 255 gates on a qubit
    q0 = (np.arange(m) // 290 % n).astype(np.int32)
    q1 = np.full(m, -1, dtype=np.int32)
    if n > 1:
        for i in (0, 288, 300, 590, 599):
            op[i], q0[i], q1[i] = W.CX, i % n, (i + 1) % n
    param = np.where(op >= 3, rng.integers(0, 7, size=m), -1).astype(np.int32)
    obs = W.obs_tfim(n) if n > 1 else W.observable([(0, 1, 0.5), (1, 0, 0.25), (1, 1, 1.0)])
    wc = W.make_circuit(n, (op, q0, q1, param), 7, obs, rng.uniform(0, 6, size=7))
    _check(api, wc, 0, [0, 6] if n < 6 else [3])


@pytest.mark.parametrize("n,m,every", [(3, 1, 1), (4, 50, 7), (5, 200, 64), (6, 400, 399), (8, 300, 50), (10, 400, 1000)])
def test_random(api, n, m, every):
    rng = np.random.default_rng(40 + n)
    wc = W.random_circuit(rng, n, m, W.obs_tfim(n))
    _check(api, wc, every, sorted(set(rng.integers(0, wc.n_params, size=6))) if wc.n_params else [])


def test_sums_flushed_between_segments(api):
    """n = 12: 4,096 tiles, 2,048 rows of sums at a time."""
    wc = W.random_circuit(np.random.default_rng(12), 12, 2600, W.obs_tfim(12))
    _check(api, wc, 500, [0, wc.n_params // 2, wc.n_params - 1])
