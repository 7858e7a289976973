"""LDS-resident evaluation from both ends, against the CPU oracle: empty and
one-sided halves, chains around the 32-record chunks, records that continue
on their pair, both weight types."""
import numpy as np
import pytest

import oracle
from paper_2502_10685_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2502_10685_amd import api as a
    return a


def _layered(seed, n, count, obs):
    """`count` CX, each with a rotation on both of its qubits behind it: about
    one record per CX."""
    rng = np.random.default_rng(seed)
    op, q0, q1, pa = [], [], [], []
    for _ in range(count):
        a, b = (int(v) for v in rng.choice(n, size=2, replace=False))
        op += [W.CX, W.RX + int(rng.integers(3)), W.RX + int(rng.integers(3))]
        q0 += [a, a, b]
        q1 += [b, -1, -1]
        pa += [-1, len(op) // 3 * 2 - 2, len(op) // 3 * 2 - 1]
    gates = (np.array(op, np.uint8), np.array(q0, np.int32), np.array(q1, np.int32), np.array(pa, np.int32))
    return W.make_circuit(n, gates, 2 * count, obs, rng.uniform(0, W.TWO_PI, size=2 * count))


# 1, 2 CX: a half without records; 62..66 and 126..130: halves of 31..33 and
# 63..65 records at the ends of one and two chunks
@pytest.mark.parametrize("n", [2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("count", [1, 2, 62, 64, 66, 126, 128, 130, 500])
def test_chain_lengths(api, n, count):
    wc = _layered([n, count], n, count, W.obs_sum_z(n))
    c = api.Circuit.from_workload(wc)
    want = oracle.expval_sv(wc)
    for _ in range(2):  # the second run finds the exchange as the first left it
        assert abs(c.evaluate().item() - want) <= 1e-12 * n
    f = api.Circuit.from_workload(wc, dtype="f32")
    # 2^-24 per rounding, at most two roundings of each weight per CX on each
    # side, and |c|_2 |r|_2 <= sqrt(n) 2^(n/2)
    bar = 2.0 ** -24 * np.sqrt(4.0 * count) * np.sqrt(n) * 2 ** (n / 2) + 1e-7
    assert abs(f.evaluate().item() - want) <= bar


@pytest.mark.parametrize("n", range(1, 8))
@pytest.mark.parametrize("m", [1, 2, 7, 40, 3000])
def test_random_circuits(api, n, m):
    wc = W.random_circuit([n, m], n, m, W.obs_tfim(n) if n > 1 else W.obs_z(1, [0]))
    got = api.Circuit.from_workload(wc).evaluate().item()
    assert abs(got - oracle.expval_sv(wc)) <= 1e-12 * 2 * n


def test_one_pair_runs_on(api):
    """Many CX and rotations on one pair: records that keep their registers."""
    wc = _layered(11, 2, 200, W.obs_z(2, [0, 1]))
    ops = (wc.op, wc.q0 + 3, np.where(wc.q1 >= 0, wc.q1 + 3, -1).astype(np.int32), wc.param)
    big = W.make_circuit(6, ops, wc.n_params, W.obs_z(6, [3, 4]), wc.theta)
    got = api.Circuit.from_workload(big).evaluate().item()
    assert abs(got - oracle.expval_sv(big)) <= 1e-12


@pytest.mark.parametrize("n", [4, 6, 7])
def test_sweep_over_more_sets_than_a_launch_holds(api, n):
    wc = W.hea_circuit(n, n, 2)
    thetas = np.random.default_rng(n).uniform(0, W.TWO_PI, size=(515, wc.n_params))
    c = api.Circuit.from_workload(wc)
    out = c.evaluate_thetas(thetas).cpu().numpy()
    for i in (0, 1, 510, 511, 512, 514):
        c.set_theta(thetas[i])
        assert out[i] == c.evaluate().item()
        assert abs(out[i] - oracle.expval_sv(wc.with_theta(thetas[i]))) <= 1e-12
