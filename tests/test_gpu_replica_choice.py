"""Which sims take the replica step, seen from what the autotuner may try: its
step is the same in every variant, the general step's is not.  Uniform graphs
take it with 16 or more replicas past the LDS bitmap (2^20 units), mixed ones
with four or more from 8192 chunks of 64 units on."""
import numpy as np
import pytest

import paper_2604_22092_amd as fs
import workloads as W

pytestmark = pytest.mark.gpu

MODEL = {"ei": W.LN_E, "ir": W.LN_I, "beta": 0.08, "dt": 0.1, "seed": 9}

CASES = [
    # name, graph, replicas, replica step
    ("uniform_r64_in_the_lds", lambda: W.random_regular_matchings(16_384, 6, 1), 64, False),
    ("uniform_r64_past_it", lambda: W.random_regular_matchings(16_386, 6, 1), 64, True),
    ("uniform_r16_past_it", lambda: W.random_regular_matchings(65_538, 6, 1), 16, True),
    ("uniform_r16_groups_of_8", lambda: W.random_regular_matchings(100_002, 6, 1), 16, True),
    ("uniform_r8_past_it", lambda: W.random_regular_matchings(131_074, 6, 1), 8, False),
    ("mixed_r4_at_8192", lambda: W.erdos_renyi(131_072, 4.0, 1), 4, True),
    ("mixed_r4_below", lambda: W.erdos_renyi(131_000, 4.0, 1), 4, False),
]


@pytest.mark.parametrize("name,graph,replicas,taken", CASES, ids=[c[0] for c in CASES])
def test_choice_and_results(name, graph, replicas, taken):
    rp, ci = graph()
    n = len(rp) - 1
    variants = 3 if n * replicas <= 1 << 20 else 2
    with fs.Graph(rp, ci) as g:
        sim = fs.Sim.from_model(g, MODEL, replicas=replicas, heavy_degree=-1)
        plain = fs.Sim.from_model(g, MODEL, replicas=replicas, heavy_degree=-1, record_rates=True)
        bins = 1 + sum(t < np.diff(rp).max() for t in (8, 12, 16, 24, 32, 64, 128, 256))
        for s in (sim, plain):
            s.seed(np.arange(100), replica=-1)
        assert sim.autotune(2, variants=True)["trials"] == bins * (1 if taken else variants)
        sim.step(12)
        plain.step(12)
        for r in (0, replicas - 1):
            np.testing.assert_array_equal(sim.history(0, 12, r), plain.history(0, 12, r))
            for a, b in zip(sim.get_state(r)[:2], plain.get_state(r)[:2]):
                np.testing.assert_array_equal(a, b)
        sim.close()
        plain.close()
