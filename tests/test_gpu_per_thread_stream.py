"""Sims and engines on hipStreamPerThread, a handle that names another stream
on every thread: state loads and reads, rates and Markovian states of graphs
of more than one transfer piece (2^17 nodes) stay in order with the kernels
that the calling thread queued."""
import numpy as np
import pytest

import paper_2604_22092_amd as fs
import workloads as W

pytestmark = pytest.mark.gpu

PER_THREAD = 2  # the value of hipStreamPerThread
N = 2 * (1 << 17) + 7


def _graph(sorted_order):
    if sorted_order:
        return W.erdos_renyi(N, 6.0, 3)
    return np.arange(N + 1, dtype=np.int32), ((np.arange(N) + 1) % N).astype(np.int32)


@pytest.mark.parametrize("sorted_order", [False, True], ids=["caller-order", "degree-sorted"])
@pytest.mark.parametrize("compact", [False, True], ids=["fp32", "compact"])
def test_states_and_rates(compact, sorted_order):
    rp, ci = _graph(sorted_order)
    model = {"ei": W.LN_E, "ir": W.LN_I, "beta": 0.2, "dt": 0.1, "seed": 3}
    storage = fs.FS_STORAGE_COMPACT if compact else fs.FS_STORAGE_FP32
    rng = np.random.default_rng(1)
    with fs.Graph(rp, ci) as g:
        sims = [fs.Sim.from_model(g, model, storage=storage, record_rates=True, stream=s) for s in (None, PER_THREAD)]
        for trial in range(3):
            st = rng.integers(0, 4, N).astype(np.int32)
            age = rng.integers(0, 300, N).astype(np.uint16) if compact else (rng.random(N) * 20).astype(np.float32)
            out = []
            for sim in sims:
                sim.set_state(st, age, step_index=0)
                got = sim.get_state()
                np.testing.assert_array_equal(got[0], st)
                np.testing.assert_array_equal(got[1], age)
                sim.step(5)
                out.append((sim.rates(), *sim.get_state()[:2], sim.history(0, 5)))
            for a, b in zip(*out):
                np.testing.assert_array_equal(a, b)
        for sim in sims:
            sim.close()


def test_markovian_states():
    rp, ci = _graph(True)
    m = {"model": "sis", "beta": 0.2, "gamma": 0.1, "seed": 5}
    rng = np.random.default_rng(2)
    with fs.Graph(rp, ci) as g:
        engines = [fs.Markov(g, m, stream=s) for s in (None, PER_THREAD)]
        for trial in range(3):
            st = (rng.random(N) < 0.3).astype(np.int32) * 2
            out = []
            for e in engines:
                e.set_state(st, step_index=0)
                np.testing.assert_array_equal(e.get_state()[0], st)
                e.step(4)
                out.append((*e.get_state()[:2], *e.history(0, 4)))
            for a, b in zip(*out):
                np.testing.assert_array_equal(a, b)
        for e in engines:
            e.close()
