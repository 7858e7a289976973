"""First passes that begin the weights themselves (chain kernels, observables
of up to 64 strings, |0...0>) against the kernels that read them from a filled
array: the same bits, alone and in batches and sweeps, for one string, repeated
strings, the longest list and one beyond, at both tile sizes, for circuits of
one pass and of many."""
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


def _obs(n, kind, rng):
    if kind == "one":
        return W.obs_random_2local(rng, n)
    if kind == "repeated":
        return W.observable([(0, 1, 0.5), (3, 1, 0.25), (0, 1, 0.125), (1 << (n - 1), 1 << (n - 1), 1.0), (3, 1, -0.75)])
    count = int(kind)
    words = rng.choice(4 ** n, size=count, replace=False)
    return W.observable([(int(w) & (2 ** n - 1), int(w) >> n, float(c)) for w, c in zip(words, rng.normal(size=count))])


@pytest.mark.parametrize("n,k,dtype", [(8, 6, "f64"), (8, 7, "f32"), (10, 7, "f64"), (10, 6, "f32"), (11, 7, "f64"),
                                       (12, 6, "f64")])
@pytest.mark.parametrize("kind", ["one", "repeated", "64", "65"])
def test_same_bits_as_a_filled_array(api, n, k, dtype, kind):
    import torch
    from paper_2502_10685_amd import _lib as L
    print(f"first pass n={n} k={k} {dtype} {kind}", flush=True)
    rng = np.random.default_rng(n + k)
    ws = [W.random_circuit(rng, n, m, _obs(n, kind, rng)) for m in (2, 25, 400)]
    cs = []
    for w in ws:
        c = api.Circuit.from_workload(w, dtype=dtype)
        c.set_option(L.PP_OPT_TILE_QUBITS, k)
        cs.append(c)
    out = torch.empty(len(cs), dtype=torch.float64, device="cuda")

    def every():
        solo = [float(c.evaluate().item()) for c in cs]
        api.evaluate_batch(cs, out)
        sweeps = [c.evaluate_thetas(torch.tensor(np.stack([w.theta, w.theta]), device="cuda")).cpu().tolist()
                  for c, w in zip(cs, ws) if w.n_params]
        return solo, out.cpu().tolist(), sweeps

    saved = L.tune_get(L.PP_TUNE_TILE_KERNEL, k)
    try:
        L.tune_set(L.PP_TUNE_TILE_KERNEL, k, 1)
        chained = every()
        L.tune_set(L.PP_TUNE_TILE_KERNEL, k, 0)
        assert every() == chained
        L.tune_set(L.PP_TUNE_TILE_KERNEL, k, 1)
        assert every() == chained
    finally:
        L.tune_set(L.PP_TUNE_TILE_KERNEL, k, saved)
    assert chained[0] == chained[1]
    for w, v in zip(ws, chained[0]):
        norm = float(np.sum(np.abs(w.obs_c)))
        assert abs(v - oracle.expval_sv(w)) <= (1e-12 if dtype == "f64" else 1e-5) * max(1.0, norm)
    for c in cs:
        c.close()
