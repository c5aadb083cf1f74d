"""The influences the Markovian engine reports for every node, also those
outside S: without I -> S a node keeps the influence it left S with until the
next full recount, whatever the order in which a step's draws and pushes ran.
Replayed one step at a time from the reported states, in steps that push, that
recount, and that leave the pushes of one crowded workgroup to the recount."""
import numpy as np
import pytest

import paper_2604_22092_amd as fs
import workloads as W

pytestmark = pytest.mark.gpu


def _recount(rp, ci, st):
    return np.add.reduceat(np.append((st[ci] == 2).astype(np.int64), 0), rp[:-1]) * (np.diff(rp) > 0)


CASES = [
    # name, graph, model, theta, p_max, inertial_max, infected first nodes (or a share of all)
    ("sir_pushes", lambda: W.erdos_renyi(60_001, 8.0, 4), "sir", 5.0, 0.6, 10**9, 0.05),
    ("seir_pushes", lambda: W.erdos_renyi(60_001, 8.0, 4), "seir", 5.0, 0.6, 10**9, 0.05),
    ("sir_both", lambda: W.erdos_renyi(60_001, 8.0, 4), "sir", 5.0, 0.6, 4000, 0.02),
    ("sir_dense", lambda: W.random_regular(20_000, 40, 2), "sir", 5.0, 0.9, 10**9, 0.2),
    # 128 nodes per workgroup, more than 4 * 600 / 157 + 64 events in the first
    ("sir_crowded", lambda: W.random_regular(20_000, 6, 3), "sir", 5.0, 5.0, 600, 128),
    ("sis_crowded", lambda: W.random_regular(20_000, 6, 3), "sis", 5.0, 5.0, 600, 128),
]


@pytest.mark.parametrize("name,graph,model,theta,p_max,most,infected", CASES, ids=[c[0] for c in CASES])
def test_influences_of_every_node(name, graph, model, theta, p_max, most, infected):
    rp, ci = graph()
    n = len(rp) - 1
    crowded = infected >= 1
    st0 = np.zeros(n, np.int32)
    if crowded:
        st0[:infected] = 2
    else:
        st0[np.random.default_rng(6).random(n) < infected] = 2
    m = {"model": model, "beta": 0.001 if crowded else 0.4, "sigma": 0.5, "gamma": 0.2, "theta": theta, "p_max": p_max,
         "tau_max": 25.0 if crowded else 2.0, "seed": 2**35 + 1}
    steps = 8
    with fs.Graph(rp, ci) as g:
        with fs.Markov(g, m, inertial_max=most) as eng:
            eng.set_state(st0, step_index=0)
            want = _recount(rp, ci, st0)
            np.testing.assert_array_equal(eng.get_state()[1], want)
            for k in range(steps):
                eng.step(1)
                st, infl, _, _ = eng.get_state()
                events = int(eng.history(k, 1)[2][0])
                if k == 0 and crowded:
                    assert 4 * most / 157 + 64 < events <= most
                now = _recount(rp, ci, st)
                want = now if model == "sis" or events > most else np.where(st == 0, now, want)
                np.testing.assert_array_equal(infl, want, err_msg=f"step {k}")
        # the same run again, its steps queued together
        with fs.Markov(g, m, inertial_max=most, steps_per_graph=4) as eng:
            eng.set_state(st0, step_index=0)
            eng.step(steps)
            got = eng.get_state()
    np.testing.assert_array_equal(got[0], st)
    np.testing.assert_array_equal(got[1], want)
