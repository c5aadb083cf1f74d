"""The Markovian step at the edges of its work split: regions of one lane, of a
partial word of nodes, of several tiles of 4096 nodes; lists longer than the
eight lanes of an event take; and steps of so many events that workgroups
leave their pushes to the recount.  Pushes and recounts must agree exactly,
and the counts must be those of the states."""
import numpy as np
import pytest

import paper_2604_22092_amd as fs
import workloads as W

pytestmark = pytest.mark.gpu


def _star_ring(n, hubs, leaves, seed):
    """A symmetric ring whose first nodes are also joined to many others."""
    rng = np.random.default_rng(seed)
    a = np.concatenate([np.arange(n), np.repeat(np.arange(hubs), leaves)])
    b = np.concatenate([(np.arange(n) + 1) % n, rng.integers(0, n, hubs * leaves)])
    return W.csr_from_edges(n, a, b)


CASES = [
    ("n7", lambda: W.complete_graph(7), "sis", 0.01),
    ("n65_hub", lambda: _star_ring(65, 1, 300, 1), "seir", 0.05),
    ("n4099_hubs", lambda: _star_ring(4099, 3, 900, 2), "sir", 0.02),
    ("tiles", lambda: W.random_regular_matchings(1_300_002, 4, 3), "sir", 0.01),
    ("er_sis", lambda: W.erdos_renyi(30_001, 8.0, 4), "sis", 5.0),
    ("er_seir", lambda: W.erdos_renyi(30_001, 8.0, 4), "seir", 5.0),
    ("many_events", lambda: W.random_regular_matchings(1_300_002, 4, 3), "sis", 0.2),
]


@pytest.mark.parametrize("name,graph,model,theta", CASES, ids=[c[0] for c in CASES])
def test_pushes_equal_recounts(name, graph, model, theta):
    rp, ci = graph()
    n = len(rp) - 1
    m = {"model": model, "beta": 0.4, "sigma": 0.5, "gamma": 0.2, "theta": theta, "p_max": 0.6, "tau_max": 2.0,
         "seed": 2**35 + 1}
    rng = np.random.default_rng(6)
    st0 = np.where(rng.random(n) < 0.05, 2, 0).astype(np.int32)
    st0[0] = 2
    steps, out = 24, []
    with fs.Graph(rp, ci) as g:
        for kw in ({"inertial_max": 10**9}, {"inertial_max": -1}, {"inertial_max": 0, "steps_per_graph": 8},
                   {"inertial_max": 3}):
            with fs.Markov(g, m, history_len=64, **kw) as eng:
                eng.set_state(st0, step_index=0)
                eng.step(steps)
                st, infl, _, t = eng.get_state()
                counts, taus, events = eng.history(0, steps)
                out.append((st, counts, taus, events, t, infl if model == "sis" else infl[st == 0]))
    for o in out[1:]:
        for x, y in zip(out[0], o):
            np.testing.assert_array_equal(x, y)
    st, counts, _, events, _, _ = out[0]
    assert np.all(counts.sum(1) == n)
    np.testing.assert_array_equal(counts[-1], np.bincount(st, minlength=4))
    # (with inertial_max = 3 a workgroup of the 256 leaves its pushes out past 64 events)
    assert events.max() > (256 * 100 if name == "many_events" else 0)
    infected = (st == 2).astype(np.int64)
    want = np.zeros(n, np.int64)
    np.add.at(want, np.repeat(np.arange(n), np.diff(rp)), infected[ci])
    np.testing.assert_array_equal(out[0][5], want if model == "sis" else want[st == 0])
