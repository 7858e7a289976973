"""The planner's schedules, from the C++ sources compiled for the host: passes
over tiles are cut into the record chain's units only where the chain runs
(n <= 14); larger circuits sweep whole groups."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2502_10685_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

DRIVER = r"""
#include <cstdio>
#include <random>
#include "plan.h"
using namespace pp;

static GateList random_gates(int n, int m, unsigned seed) {
    std::mt19937 r(seed);
    GateList g;
    g.n = n;
    g.m = m;
    int p = 0;
    for (int i = 0; i < m; ++i) {
        const bool rot = r() & 1;
        const uint8_t op = (uint8_t)(r() % 3 + (rot ? 3 : 0));
        const int a = (int)(r() % n), b = (a + 1 + (int)(r() % (n - 1))) % n;
        g.op.push_back(op);
        g.q0.push_back(a);
        g.q1.push_back(op == 2 ? b : -1);
        g.param.push_back(rot ? p++ : -1);
    }
    g.n_params = p;
    return g;
}

static int sweeps(const DensePlan &P) {
    int s = 0;
    for (size_t i = 0; i < P.ops.size(); ++s) i += P.ops[i].kind == DOP_GROUP ? 1 + P.ops[i].ngates : 1;
    return s;
}

int main() {
    for (int n = 13; n <= 16; ++n)
        for (int k = 6; k <= 7; ++k) {
            const GateList g = random_gates(n, 3000, 7u * n + k);
            PlanOptions o;
            o.segments = false;
            const DensePlan whole = plan_dense_opts(g, k, 2, o);
            o.chain = chain_tiles(k, n, false);
            const DensePlan P = plan_dense_opts(g, k, 2, o);
            const std::string bad = plan_check(P, n);
            std::printf("%d %d %d %d %d %s\n", n, k, (int)o.chain, sweeps(whole), sweeps(P), bad.empty() ? "ok" : bad.c_str());
        }
    return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("plan")
    (d / "driver.cpp").write_text(DRIVER)
    flags = ["-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-w", "-I", CSRC, "-c"]
    for src in (os.path.join(CSRC, "plan.cpp"), str(d / "driver.cpp")):
        subprocess.run([HIPCC, *flags, src, "-o", str(d / (os.path.basename(src) + ".o"))], check=True)
    subprocess.run([HIPCC, "-o", str(d / "driver"), str(d / "plan.cpp.o"), str(d / "driver.cpp.o")], check=True)
    return str(d / "driver")


def test_chain_units_only_where_the_chain_runs(driver):
    rows = [ln.split() for ln in subprocess.run([driver], check=True, capture_output=True, text=True).stdout.splitlines()]
    assert len(rows) == 8
    for n, k, chain, whole, planned, ok in rows:
        assert ok == "ok" and int(chain) == (int(n) <= 14)
        assert int(planned) == int(whole) if int(n) > 14 else int(planned) > int(whole)
