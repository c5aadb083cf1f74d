"""A change of bins, of the step variant or an autotune that runs out of memory
at any of its allocations leaves the sim stepping as it did, and the same call
succeeds afterwards."""
import ctypes

import numpy as np
import pytest

import paper_2604_22092_amd as fs
import workloads as W

pytestmark = pytest.mark.gpu

MODEL = {"ei": ("erlang", 3, 1.0), "ir": ("weibull", 2.0, 6.0), "beta": 0.1, "dt": 0.1, "seed": 5}


class _Failing:
    """The library's allocator hook: device memory, but for one request."""

    def __init__(self, fail_at):
        self.left, self.failed = fail_at, False

    def alloc(self, nbytes):
        if self.left == 0:
            self.failed = True
            self.left = -1
            return 0
        self.left -= 1
        p = ctypes.c_void_p()
        assert fs.lib().hipMalloc(ctypes.byref(p), ctypes.c_size_t(nbytes)) == 0
        return p.value

    @staticmethod
    def free(p):
        fs.lib().hipFree(ctypes.c_void_p(p))

    def __enter__(self):
        fs.set_allocator(self.alloc, self.free)
        return self

    def __exit__(self, *exc):
        fs.set_allocator()


def _weighted(graph, seed):
    rp, ci = graph
    return rp, ci, np.random.default_rng(seed).random(len(ci)).astype(np.float32)


def _sim(g, n, replicas, **kw):
    sim = fs.Sim.from_model(g, MODEL, replicas=replicas, **kw)
    st = np.random.default_rng(4).choice(4, size=n, p=[0.8, 0.05, 0.1, 0.05]).astype(np.int32)
    for r in range(replicas):
        sim.set_state(st, np.zeros(n, np.float32), r, step_index=0)
    return sim


CASES = [
    # name, graph, replicas, calls in turn, the allocations that fail
    ("replica_step_left", lambda: W.barabasi_albert(40_000, 6, 5), 16, lambda s: s.set_bins(-1), range(20)),
    ("replica_step_bins", lambda: W.barabasi_albert(40_000, 6, 5), 16, lambda s: s.set_bins(12), range(20)),
    ("pushed_bins", lambda: W.barabasi_albert(20_000, 5, 5), 1, lambda s: s.set_bins(12), range(20)),
    ("segment_bins", lambda: _weighted(W.barabasi_albert(20_000, 5, 5), 1), 2, lambda s: s.set_bins(12), range(20)),
    ("autotune", lambda: W.barabasi_albert(20_000, 5, 5), 2, lambda s: s.autotune(3, variants=True),
     [0, 3, 9, 13, 14, 15, 20, 21, 25, 32, 40, 51]),
    ("autotune_replicas", lambda: W.barabasi_albert(40_000, 6, 5), 16, lambda s: s.autotune(3, variants=True),
     [0, 5, 9, 13, 14, 17, 20, 23, 30]),
]


@pytest.mark.parametrize("name,graph,replicas,call,at", CASES, ids=[c[0] for c in CASES])
def test_a_failed_call_changes_nothing(name, graph, replicas, call, at):
    spec = graph()
    n = len(spec[0]) - 1
    with fs.Graph(*spec) as g:
        ref, sim = _sim(g, n, replicas), _sim(g, n, replicas, steps_per_graph=2)
        bins, variant = sim.bins(), sim.variant()
        sim.step(2)
        ref.step(2)
        k, failures = 2, 0
        for i in at:
            print(name, "allocation", i, flush=True)
            with _Failing(i) as hook:
                try:
                    call(sim)
                except fs.FsError:
                    assert hook.failed
            if not hook.failed:
                break
            failures += 1
            assert sim.bins() == bins and sim.variant() == variant
            sim.step(3)
            ref.step(3)
            k += 3
            for r in (0, replicas - 1):
                np.testing.assert_array_equal(sim.history(k - 3, 3, r), ref.history(k - 3, 3, r))
        assert failures >= 3
        call(sim)
        sim.step(3)
        ref.step(3)
        for r in (0, replicas - 1):
            np.testing.assert_array_equal(sim.history(k, 3, r), ref.history(k, 3, r))
            for a, b in zip(sim.get_state(r)[:2], ref.get_state(r)[:2]):
                np.testing.assert_array_equal(a, b)
        sim.close()
        ref.close()


def test_a_failed_join_changes_nothing():
    """Joining a batch moves a packed, summary-stepped sim to plain columns and
    the streaming step."""
    rp, ci = W.erdos_renyi(2**20 + 1, 3.0, 1)
    n = len(rp) - 1
    with fs.Graph(rp, ci) as g:
        ref, sim = _sim(g, n, 1), _sim(g, n, 1)
        assert sim.variant() == "summary"
        k, failures = 0, 0
        with fs.Batch() as b:
            for i in range(20):
                print("allocation", i, flush=True)
                with _Failing(i) as hook:
                    try:
                        b.add(sim)
                    except fs.FsError:
                        assert hook.failed
                if not hook.failed:
                    break
                failures += 1
                assert b.size() == 0
                sim.step(2)
                ref.step(2)
                k += 2
                np.testing.assert_array_equal(sim.history(k - 2, 2), ref.history(k - 2, 2))
            assert failures >= 3 and b.size() == 1
            b.step(3)
            ref.step(3)
            np.testing.assert_array_equal(sim.history(k, 3), ref.history(k, 3))
            np.testing.assert_array_equal(sim.get_state()[0], ref.get_state()[0])
            b.remove(sim)
        sim.close()
        ref.close()
