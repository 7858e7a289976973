"""FP32 circuits that fit one workgroup's LDS are propagated in doubles and
rounded where the weights leave the chip, once.  So the density matrix is off
by at most half a unit in the last place of each weight, 2^-24 of its norm (it
is a linear, norm-preserving map of the weights, computed in FP64), and <O> of
up to 5 qubits (both ends in one workgroup) agrees with FP64 to 1e-12.  With 6
and 7 qubits the two ends' vectors c and r are rounded when they meet: |<O>| is
off by at most (2^-24 + 2^-24) |c| |r| + 1e-12, with |r| = 2^(n/2) and |c| the
2-norm of the observable."""
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


def _circuits(n):
    rng = np.random.default_rng(40 + n)
    gates, p = W.chain_zxz_gates(n, 12, 6)
    yield W.make_circuit(n, gates, p, W.obs_tfim(n), rng.uniform(0.0, 6.28, size=p))
    yield W.random_circuit(rng, n, 2500, W.obs_tfim(n))


@pytest.mark.parametrize("n", [2, 3, 4, 5, 6, 7])
def test_rounded_once(api, n):
    print(f"f32 rounding n={n}", flush=True)
    for w in _circuits(n):
        rho, ev = [], []
        for dtype in ("f64", "f32"):
            c = api.Circuit.from_workload(w, dtype=dtype)
            rho.append(c.density_matrix().cpu().numpy())
            ev.append(float(c.evaluate().item()))
            c.close()
        assert np.linalg.norm(rho[1] - rho[0]) <= 2.0 ** -24 * (1 + 1e-9) * np.linalg.norm(rho[0])
        meet = 2.0 ** -23 * np.linalg.norm(w.obs_c) * 2.0 ** (n / 2) if n > 5 else 0.0
        assert abs(ev[1] - ev[0]) <= meet + 1e-12
