"""Passes over 7-qubit tiles run as record chains: against the CPU oracle, and
bit for bit against one workgroup per tile, which runs the same schedule."""
import numpy as np
import pytest

import oracle
from paper_2502_10685_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2502_10685_amd import api as a
    return a


def _on(qubits, n, m, seed):
    """m random gates on `qubits` of an n-qubit register, then one CX between
    the lowest of them and a qubit outside."""
    wc = W.random_circuit([seed, m], len(qubits), m)
    q = np.array(qubits, np.int32)
    q0, q1 = q[wc.q0], np.where(wc.q1 >= 0, q[wc.q1], -1)
    out = next(i for i in range(n) if i not in qubits)
    gates = (np.append(wc.op, W.CX).astype(np.uint8), np.append(q0, qubits[0]).astype(np.int32),
             np.append(q1, out).astype(np.int32), np.append(wc.param, -1).astype(np.int32))
    return W.make_circuit(n, gates, wc.n_params, W.obs_sum_z(n), wc.theta)


def _check(api, wc, dtype, tol):
    from paper_2502_10685_amd import _lib as L
    vals = []
    old = L.tune_get(L.PP_TUNE_TILE_KERNEL, 7)
    try:
        for variant in (0, 1):
            L.tune_set(L.PP_TUNE_TILE_KERNEL, 7, variant)
            c = api.Circuit.from_workload(wc, engine="dense", tile_qubits=7, dtype=dtype)
            vals.append([c.evaluate().item(), c.evaluate().item()])
            c.close()
    finally:
        L.tune_set(L.PP_TUNE_TILE_KERNEL, 7, old)
    assert vals[0] == vals[1] and vals[1][0] == vals[1][1], vals
    assert abs(vals[1][0] - oracle.expval_sv(wc)) <= tol


# one, two and few gates (passes of two records), then passes within a chunk
@pytest.mark.parametrize("n", [8, 9, 11])
@pytest.mark.parametrize("m", [1, 2, 5, 60, 1500])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_random(api, n, m, dtype):
    wc = W.random_circuit([7, n, m], n, m, W.obs_tfim(n))
    # FP32: 2^-24 per rounding, |c|_2 |r|_2 <= sqrt(2n) 2^(n/2)
    bar = 1e-12 * 2 * n if dtype == "f64" else 2.0 ** -24 * np.sqrt(m) * np.sqrt(2 * n) * 2 ** (n / 2)
    _check(api, wc, dtype, bar)


# all gates on seven qubits: one pass of many chunks of 32 records; on the two
# lowest only: no record avoids them
@pytest.mark.parametrize("qubits", [[0, 1, 2, 3, 4, 5, 6], [0, 1, 3, 5, 6, 7, 8], [0, 1]])
@pytest.mark.parametrize("m", [150, 190, 210, 400, 900])
def test_long_passes(api, qubits, m):
    _check(api, _on(qubits, 10, m, 3), "f64", 1e-11)


def test_more_tiles_than_workgroups(api):
    wc = W.random_circuit([7, 12], 12, 400, W.obs_z(12, [0, 11]))
    _check(api, wc, "f64", 1e-12)


def test_batch_of_mixed_sizes(api):
    import torch
    wcs = [W.random_circuit([70, i], 8 + i % 5, 100 + 37 * i) for i in range(15)]
    cs = [api.Circuit.from_workload(w, tile_qubits=7) for w in wcs]
    solo = torch.stack([c.evaluate() for c in cs])
    both = api.evaluate_batch(cs)
    assert torch.equal(solo, both)
    for v, w in zip(both.tolist(), wcs):
        assert abs(v - oracle.expval_sv(w)) <= 1e-12
