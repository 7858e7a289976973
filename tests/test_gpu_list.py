"""Rotations on the string list (one kernel per rotation, pairs found through
a hash table): the string set, the weights, the dropped weight and <O> against
a plain dictionary that merges and cuts after every rotation, from one string
to lists beyond one tile per workgroup, up to 64 qubits, with repeated
observable strings, weight cuts, closing Clifford runs and the capacity's last
string.

Tolerances: a weight goes through at most m roundings of sums of two products
(4 units in the last place of 1.0 each): 4 m 2^-53 in FP64, 4 m 2^-24 in
FP32, doubled for the angles' sine and cosine."""
import math
import sys

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


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _clifford(op, a, b, x, z):
    bit = lambda w, q: (w >> q) & 1
    xa, za = bit(x, a), bit(z, a)
    if op == W.H:
        f = (xa ^ za) << a
        return x ^ f, z ^ f, xa & za
    if op == W.S:
        return x, z ^ (xa << a), xa & (za ^ 1)
    xb, zb = bit(x, b), bit(z, b)
    return x ^ (xa << b), z ^ (zb << a), xa & zb & (xb ^ za ^ 1)


def _child(op, q, x, z):
    xb, zb, bit = (x >> q) & 1, (z >> q) & 1, 1 << q
    if op == W.RX:
        return (bit, 0, -1.0 if xb else 1.0) if zb else None
    if op == W.RY:
        return (bit, bit, 1.0 if xb else -1.0) if xb ^ zb else None
    return (0, bit, 1.0 if zb else -1.0) if xb else None


def _propagate(wc, eps, wmax, dtype):
    """(merged strings {(x, z): weight}, dropped weight)"""
    ft = np.float64 if dtype == "f64" else np.float32
    heavy = lambda x, z: bin(x | z).count("1") > wmax
    terms = [(int(x), int(z), ft(c)) for x, z, c in zip(wc.obs_x, wc.obs_z, wc.obs_c)]
    dropped, pending = 0.0, True

    def merge(ts):
        out, lost = {}, 0.0
        for x, z, c in ts:
            out[(x, z)] = out.get((x, z), 0.0) + float(c)
        for (x, z), c in list(out.items()):
            if heavy(x, z) or not abs(c) >= eps:
                lost += abs(c)
                del out[(x, z)]
        return [(x, z, ft(c)) for (x, z), c in out.items()], lost

    for g in range(wc.m - 1, -1, -1):
        op, a, b = int(wc.op[g]), int(wc.q0[g]), int(wc.q1[g])
        if op <= 2:
            ts = [(_clifford(op, a, b, x, z), c) for x, z, c in terms]
            terms = [(x, z, -c if neg else c) for (x, z, neg), c in ts]
            pending = True
            continue
        cs, sn = math.cos(wc.theta[wc.param[g]]), math.sin(wc.theta[wc.param[g]])
        new, kids = [], []
        for x, z, c in terms:
            k = _child(op, a, x, z)
            if k is None:
                new.append((x, z, c))
                continue
            new.append((x, z, ft(float(c) * cs)))
            kx, kz = x ^ k[0], z ^ k[1]
            if heavy(kx, kz):
                dropped += abs(float(c) * k[2] * sn)
            else:
                kids.append((kx, kz, ft(float(c) * k[2] * sn)))
        terms, lost = merge(new + kids)
        dropped += lost
        pending = False
    if pending:
        terms, lost = merge(terms)
        dropped += lost
    return {(x, z): float(c) for x, z, c in terms}, dropped


def _random(n, m, seed, obs, tail):
    rng = np.random.default_rng(seed)
    wc = W.random_circuit(rng, n, m, obs)
    if tail:  # the first gates are met last: a closing Clifford run
        wc.op[:tail], wc.q0[:tail], wc.param[:tail] = W.CX, np.arange(tail) % (n - 1), -1
        wc.q1[:tail] = wc.q0[:tail] + 1
    return wc


def _repeated(n):
    return W.observable([(0, 1, 0.5), (3, 1, 0.25), (0, 1, 0.125), (1 << (n - 1), 1 << (n - 1), 1.0), (3, 1, -0.25)])


@pytest.mark.parametrize("n,m,eps,wmax,obs,tail,dtype", [
    (4, 60, 0.0, 64, "tfim", 0, "f64"),
    (8, 1, 0.0, 64, "tfim", 1, "f64"),         # Clifford gates alone
    (33, 110, 1e-4, 64, "tfim", 3, "f64"),
    (64, 260, 2e-2, 64, "tfim", 0, "f64"),
    (40, 300, 0.0, 3, "repeated", 2, "f64"),   # repeated strings, a weight cut
    (12, 150, 1e-3, 5, "tfim", 0, "f32"),
    (48, 300, 1e-2, 64, "repeated", 0, "f32"),
])
def test_against_dictionary(api, n, m, eps, wmax, obs, tail, dtype):
    from paper_2502_10685_amd import _lib as L
    _say(f"list n={n} m={m} eps={eps} wmax={wmax} {obs} {dtype}")
    wc = _random(n, m, 70 + n, _repeated(n) if obs == "repeated" else W.obs_tfim(n), tail)
    ref, dropped = _propagate(wc, eps, wmax, dtype)
    c = api.Circuit.from_workload(wc, engine="sparse", dtype=dtype, max_terms=1 << 18)
    c.set_option(L.PP_OPT_SPARSE_FRAME, 0)
    if eps or wmax < 64:
        c.set_truncation(eps, wmax)
    tol = 8 * m * (2.0 ** -53 if dtype == "f64" else 2.0 ** -24)
    evs = []
    for _ in range(2):
        evs.append(float(c.evaluate().item()))
        assert c.stats()["final_terms"] == len(ref) and not c.stats()["overflow"]
        x, z, v = c.terms(capacity=1 << 18)
        keys = [(int(b), int(a)) for a, b in zip(x, z)]
        assert keys == sorted((zz, xx) for xx, zz in ref), "string sets differ"
        assert max([abs(w - ref[(k[1], k[0])]) for k, w in zip(keys, v)], default=0.0) <= tol
        assert abs(evs[-1] - sum(w for (xx, _), w in ref.items() if xx == 0)) <= tol * max(1, len(ref))
        assert abs(c.truncation_dropped() - dropped) <= tol * max(1.0, dropped) * max(1, len(ref))
    assert evs[0] == evs[1]
    c.close()


def _product(n, theta):
    gates = ([W.RX] * n, list(range(n)), [-1] * n, list(range(n)))
    arr = [np.array(a, dtype=t) for a, t in zip(gates, (np.uint8, np.int32, np.int32, np.int32))]
    return W.make_circuit(n, tuple(arr), n, W.obs_z(n, range(n)), theta)


@pytest.mark.parametrize("n,dtype", [(21, "f64"), (20, "f32")])
def test_lists_beyond_one_tile_per_workgroup(api, n, dtype):
    """Z...Z under an RX on every qubit: 2^n strings, <O> = prod cos."""
    from paper_2502_10685_amd import _lib as L
    _say(f"list product n={n} {dtype}")
    theta = np.random.default_rng(n).uniform(0.1, 0.6, size=n)
    c = api.Circuit.from_workload(_product(n, theta), engine="sparse", dtype=dtype, max_terms=1 << n)
    c.set_option(L.PP_OPT_SPARSE_FRAME, 0)
    ev = float(c.evaluate().item())
    assert c.stats()["final_terms"] == 1 << n and c.stats()["term_updates"] == (1 << n) - 1
    x, z, v = c.terms(capacity=1 << n)
    tol = 8 * n * (2.0 ** -53 if dtype == "f64" else 2.0 ** -24)
    assert abs(ev - np.prod(np.cos(theta))) <= tol
    assert np.array_equal(x, np.arange(1 << n, dtype=np.uint64)) and np.all(z == (1 << n) - 1)
    ref = np.ones(1)
    for t in theta:  # qubit q is bit q of x
        ref = np.concatenate([ref * math.cos(t), ref * math.sin(t)])
    assert float(np.max(np.abs(v - ref))) <= tol
    c.close()


@pytest.mark.parametrize("n", [4, 10])
def test_capacity_edge(api, n):
    """The capacity counts the strings before equal ones are merged: twice
    max_terms of them fit, one more does not."""
    from paper_2502_10685_amd import _lib as L
    _say(f"list capacity n={n}")
    theta = np.full(n, 0.3)
    for cap, fits in ((1 << (n - 1), True), ((1 << (n - 1)) - 1, False)):
        c = api.Circuit.from_workload(_product(n, theta), engine="sparse", max_terms=cap)
        c.set_option(L.PP_OPT_SPARSE_FRAME, 0)
        ev = float(c.evaluate().item())
        assert bool(c.stats()["overflow"]) is not fits
        assert math.isnan(ev) is not fits
        c.close()


def test_graph_replays(api):
    from paper_2502_10685_amd import _lib as L
    wc = W.random_circuit(np.random.default_rng(8), 34, 90, W.obs_tfim(34))
    c = api.Circuit.from_workload(wc, engine="sparse", max_terms=1 << 18)
    c.set_truncation(1e-3, 64)
    eager = float(c.evaluate().item())
    c.set_option(L.PP_OPT_USE_GRAPH, 1)
    for _ in range(3):
        assert float(c.evaluate().item()) == eager
        assert c.stats()["final_terms"] == len(c.terms(capacity=1 << 18)[0])
    c.close()
