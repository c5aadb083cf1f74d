"""State loads and reads move in pieces of 2^17 nodes: round trips and refused
loads at the edges of a piece, in the caller's order and on a degree-sorted
graph, for both storages, several replicas and the Markovian engine."""
import numpy as np
import pytest

import paper_2604_22092_amd as fs
import workloads as W

pytestmark = pytest.mark.gpu

PIECE = 1 << 17
MODEL = {"ei": W.LN_E, "ir": W.LN_I, "beta": 0.1, "dt": 0.1, "seed": 3}


def _graph(n, sorted_order):
    """A ring, or (for a degree-sorted internal order) a ring whose node i also
    lists node 0 when i is a multiple of 3."""
    if not sorted_order:
        return np.arange(n + 1, dtype=np.int32), ((np.arange(n) + 1) % n).astype(np.int32)
    extra = (np.arange(n) % 3 == 0).astype(np.int64)
    rp = np.concatenate([[0], np.cumsum(1 + extra)])
    ci = np.zeros(rp[-1], np.int32)
    ci[rp[:-1]] = (np.arange(n) + 1) % n
    return rp.astype(np.int32), ci


def _state(n, compact, seed):
    rng = np.random.default_rng(seed)
    st = rng.integers(0, 4, n).astype(np.int32)
    if compact:
        return st, rng.integers(0, 65536, n).astype(np.uint16)
    age = rng.random(n).astype(np.float32) * 50
    age[0], age[-1] = np.float32(-0.0), np.finfo(np.float32).max
    return st, age


@pytest.mark.parametrize("sorted_order", [False, True], ids=["caller-order", "degree-sorted"])
@pytest.mark.parametrize("compact", [False, True], ids=["fp32", "compact"])
@pytest.mark.parametrize("n", [1, 2, PIECE - 1, PIECE, PIECE + 1, 2 * PIECE + 7, 9 * PIECE + 1])
def test_state_round_trip(n, compact, sorted_order):
    rp, ci = _graph(n, sorted_order)
    storage = fs.FS_STORAGE_COMPACT if compact else fs.FS_STORAGE_FP32
    with fs.Graph(rp, ci) as g:
        sim = fs.Sim.from_model(g, MODEL, replicas=2, storage=storage)
        want = [_state(n, compact, r) for r in range(2)]
        for r in range(2):
            sim.set_state(*want[r], replica=r, step_index=4)
        bad = want[0][0].copy()
        bad[-1] = 4
        with pytest.raises(fs.FsError):
            sim.set_state(bad, want[1][1], replica=0)
        bad[-1] = -1
        with pytest.raises(fs.FsError):
            sim.set_state(bad, want[1][1], replica=0)
        if not compact:
            for v in (np.nan, np.inf, -1.0):
                age = want[1][1].copy()
                age[-1] = v
                with pytest.raises(fs.FsError):
                    sim.set_state(want[1][0], age, replica=0)
        for r in range(2):
            st, age, k = sim.get_state(r)
            assert k == 4
            np.testing.assert_array_equal(st, want[r][0])
            np.testing.assert_array_equal(age, want[r][1])
            assert sim.counts(r).tolist() == np.bincount(want[r][0], minlength=4).tolist()
        sim.close()


@pytest.mark.parametrize("sorted_order", [False, True], ids=["caller-order", "degree-sorted"])
def test_markov_state_round_trip(sorted_order):
    n = 2 * PIECE + 7
    rp, ci = _graph(n, sorted_order)
    st = np.random.default_rng(5).integers(0, 4, n).astype(np.int32)
    with fs.Graph(rp, ci) as g:
        eng = fs.Markov(g, {"model": "seir", "beta": 0.2, "sigma": 0.3, "gamma": 0.1})
        eng.set_state(st, step_index=2, elapsed=1.5)
        bad = st.copy()
        bad[-1] = 7
        with pytest.raises(fs.FsError):
            eng.set_state(bad)
        got, infl, k, t = eng.get_state()
        eng.close()
    assert (k, t) == (2, 1.5)
    np.testing.assert_array_equal(got, st)
    want = np.add.reduceat((st[ci] == 2).astype(np.int32), rp[:-1])
    np.testing.assert_array_equal(infl, want)


def test_history_longer_than_a_buffer():
    n, steps = 8, 60_000  # 16 bytes a row: more than one pinned buffer holds
    rp, ci = _graph(n, False)
    with fs.Graph(rp, ci) as g:
        sim = fs.Sim.from_model(g, MODEL, replicas=2, steps_per_graph=1000, history_len=steps)
        sim.seed([0, 3], replica=-1)
        sim.step(steps + 500)
        h = sim.history(500, steps, 1)
        np.testing.assert_array_equal(sim.history(500 + steps - 9, 9, 1), h[-9:])
        sim.close()
    assert np.all(h.sum(1) == n)
    assert np.all(np.diff(h[:, 0]) <= 0) and np.all(np.diff(h[:, 3]) >= 0)
