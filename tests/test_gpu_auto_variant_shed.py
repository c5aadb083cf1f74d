"""The automatic step variant of shedding sims past the LDS bitmap: with binned
rows the summary only from 5 * 2^19 units on, and the same results either way."""
import numpy as np
import pytest

import paper_2604_22092_amd as fs
import workloads as W

pytestmark = pytest.mark.gpu

MODEL = {"ei": ("erlang", 3, 1.0), "ir": ("weibull", 2.0, 6.0), "beta": 0.3, "dt": 0.1, "seed": 5,
         "shed": ("density", ("lognormal", 0.9, 0.5), 4.0)}

CASES = [
    # name, graph, replicas, bins, chosen variant
    ("er", lambda: W.erdos_renyi(2**20 + 1, 3.0, 1), 1, 0, "summary"),
    ("ba", lambda: W.barabasi_albert(1_060_000, 2, 1), 1, 0, "stream"),
    ("ba_unbinned", lambda: W.barabasi_albert(1_060_000, 2, 1), 1, -1, "summary"),
    ("ba_two_replicas", lambda: W.barabasi_albert(530_000, 2, 1), 2, 0, "stream"),
    ("ba_large", lambda: W.barabasi_albert(5 * 2**18, 2, 1), 2, 0, "summary"),
]


@pytest.mark.parametrize("name,graph,replicas,bins,chosen", CASES, ids=[c[0] for c in CASES])
def test_choice_and_results(name, graph, replicas, bins, chosen):
    rp, ci = graph()
    n = len(rp) - 1
    st = np.random.default_rng(4).choice(4, size=n, p=[0.8, 0.05, 0.1, 0.05]).astype(np.int32)
    outs = []
    with fs.Graph(rp, ci) as g:
        for variant in (fs.VARIANT_AUTO, fs.VARIANT_STREAM, fs.VARIANT_SUMMARY):
            sim = fs.Sim.from_model(g, MODEL, replicas=replicas, heavy_degree=bins, variant=variant)
            if variant == fs.VARIANT_AUTO:
                assert sim.variant() == chosen
            for r in range(replicas):
                sim.set_state(st, np.zeros(n, np.float32), r, step_index=0)
            sim.step(6)
            outs.append([(*sim.get_state(r)[:2], sim.history(0, 6, r)) for r in range(replicas)])
            sim.close()
    for o in outs[1:]:
        for a, b in zip(outs[0], o):
            for x, y in zip(a, b):
                np.testing.assert_array_equal(x, y)
