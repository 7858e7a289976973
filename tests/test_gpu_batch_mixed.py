"""Batches that hold DENSE circuits of more than 14 qubits (whose passes run one
workgroup per tile) beside smaller ones of the same tile size (whose first
passes begin their weights): every value equals the circuit's own evaluation
bit for bit, in both orders, again with other angles, and captured."""
import numpy as np
import pytest

from paper_2502_10685_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("k,sizes", [(0, [(15, 60), (8, 300), (9, 200), (10, 120)]),
                                     (7, [(15, 60), (10, 700), (11, 200), (14, 80)])])
def test_batch_past_14_qubits_beside_smaller_circuits(k, sizes, graph):
    import torch
    from paper_2502_10685_amd import _lib as L
    from paper_2502_10685_amd import api
    assert torch.cuda.is_available(), "GPU tests need a visible HIP device"
    print(f"mixed batch k={k} graph={graph}", flush=True)
    rng = np.random.default_rng(150 + k)
    ws = [W.random_circuit(rng, n, m, W.obs_tfim(n)) for n, m in sizes]

    def made(w, graph):
        c = api.Circuit.from_workload(w, dtype="f32", engine="dense", tile_qubits=k)
        c.set_option(L.PP_OPT_USE_GRAPH, graph)
        return c

    thetas = [[w.theta for w in ws], [w.theta[::-1].copy() for w in ws]]
    want = []
    for i, w in enumerate(ws):
        c = made(w, 0)
        want.append([])
        for t in thetas:
            c.set_theta(t[i])
            want[-1].append(float(c.evaluate().item()))
        c.close()
    assert len({v for pair in want for v in pair}) == 2 * len(ws)
    order = list(range(len(ws)))
    for o in (order, order[::-1]):
        cs = [made(ws[i], graph) for i in o]
        out = torch.empty(len(cs), dtype=torch.float64, device="cuda")
        for turn in (0, 1, 1, 0):
            for c, i in zip(cs, o):
                c.set_theta(thetas[turn][i])
            api.evaluate_batch(cs, out)
            assert out.cpu().tolist() == [want[i][turn] for i in o]
        for c in cs:
            c.close()
