"""The counts of a launch sequence at the edges of the reduce's tiles: sequences
of one slot, of as many as one pass takes (1024 / 4R, one per thread) and of
several passes, over rings shorter and longer than the sequence, against the
counts of the states after every step."""
import numpy as np
import pytest

import paper_2604_22092_amd as fs
import workloads as W

pytestmark = pytest.mark.gpu

MODEL = {"ei": ("erlang", 3, 1.0), "ir": ("weibull", 2.0, 6.0), "beta": 0.3, "dt": 0.1, "seed": 5}


@pytest.mark.parametrize("replicas", [1, 2, 16, 32, 64])
@pytest.mark.parametrize("ring", [0, 37], ids=["ring1024", "ring37"])
def test_counts_of_long_sequences(replicas, ring):
    n = 700
    rp, ci = W.erdos_renyi(n, 6.0, 3)
    one = 1024 // (4 * replicas)
    with fs.Graph(rp, ci) as g:
        ref = fs.Sim.from_model(g, MODEL, replicas=replicas)
        ref.seed(np.arange(20), replica=-1)
        want = []
        top = 4 * one + 3
        for _ in range(2 * top):
            ref.step(1)
            want.append([ref.counts(r) for r in (0, replicas - 1)])
        ref.close()
        want = np.array(want)
        for length in sorted({1, 2, one - 1, one, one + 1, 4 * one, top} - {0}):
            sim = fs.Sim.from_model(g, MODEL, replicas=replicas, steps_per_graph=length, history_len=ring)
            sim.seed(np.arange(20), replica=-1)
            sim.step(2 * length)  # two replays
            kept = min(2 * length, ring or 1024)
            for i, r in enumerate((0, replicas - 1)):
                np.testing.assert_array_equal(sim.history(2 * length - kept, kept, r),
                                              want[2 * length - kept:2 * length, i], err_msg=f"{length} {r}")
            sim.close()
