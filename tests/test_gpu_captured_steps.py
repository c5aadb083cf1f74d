"""Steps queued while the caller captures the sim's stream into a graph of its
own: every replay steps from the state the sim holds then, also one that was
loaded after the capture, and the counts it records are those of that state."""
import ctypes

import numpy as np
import pytest

import paper_2604_22092_amd as fs
import workloads as W

pytestmark = pytest.mark.gpu

MODEL = {"ei": ("erlang", 3, 1.0), "ir": ("weibull", 2.0, 6.0), "beta": 0.2, "dt": 0.1, "seed": 5}
THREAD_LOCAL = 1  # hipStreamCaptureModeThreadLocal


class _Capture:
    """A stream and graphs of work queued on it (the library's own HIP runtime)."""

    def __init__(self):
        self.stream = ctypes.c_void_p()
        self._ok("hipStreamCreateWithFlags", ctypes.byref(self.stream), ctypes.c_uint(1))

    def _ok(self, name, *args):
        err = getattr(fs.lib(), name)(*args)
        assert err == 0, f"{name}: {err}"

    def graph(self, queue):
        g, x = ctypes.c_void_p(), ctypes.c_void_p()
        self._ok("hipStreamBeginCapture", self.stream, ctypes.c_int(THREAD_LOCAL))
        queue()
        self._ok("hipStreamEndCapture", self.stream, ctypes.byref(g))
        self._ok("hipGraphInstantiate", ctypes.byref(x), g, None, None, ctypes.c_size_t(0))
        self._ok("hipGraphDestroy", g)
        return x

    def launch(self, x):
        self._ok("hipGraphLaunch", x, self.stream)

    def close(self, *graphs):
        for x in graphs:
            self._ok("hipGraphExecDestroy", x)
        self._ok("hipStreamDestroy", self.stream)


def _states(n, replicas, seed):
    rng = np.random.default_rng(seed)
    return [rng.choice(4, size=n, p=[0.7, 0.1, 0.1, 0.1]).astype(np.int32) for _ in range(replicas)]


def _load(sim, states, k):
    for r, st in enumerate(states):
        sim.set_state(st, np.zeros(len(st), np.float32), r, step_index=k)


CASES = [
    ("regular_r1", lambda: W.random_regular(5001, 6, 1), 1),
    ("er_r4", lambda: W.erdos_renyi(5001, 6.0, 1), 4),
    ("replica_step_r16", lambda: W.erdos_renyi(33_001, 8.0, 1), 16),
]


@pytest.mark.parametrize("batched", [False, True], ids=["alone", "batch"])
@pytest.mark.parametrize("name,graph,replicas", CASES, ids=[c[0] for c in CASES])
def test_replays_after_state_loads(name, graph, replicas, batched):
    rp, ci = graph()
    n = len(rp) - 1
    c = _Capture()
    with fs.Graph(rp, ci) as g:
        kw = {"replicas": replicas, "variant": fs.VARIANT_STREAM if batched else fs.VARIANT_AUTO}
        sim = fs.Sim.from_model(g, MODEL, **({} if batched else {"stream": c.stream.value}), **kw)
        ref = fs.Sim.from_model(g, MODEL, **kw)
        batch = fs.Batch(stream=c.stream.value) if batched else None
        if batched:
            batch.add(sim)
        step = batch.step if batched else sim.step
        sim.seed(np.arange(9), replica=-1)
        step(3)
        exe = c.graph(lambda: step(4))
        for trial in range(4):
            k = 20 * trial
            states = _states(n, replicas, trial)
            _load(sim, states, k)
            c.launch(exe)      # steps k .. k + 3 (the sim still reports step k)
            if trial % 2:
                c.launch(exe)  # and 4 more from there
            step(8 if trial % 2 else 4)
            _load(ref, states, k)
            ref.step(16 if trial % 2 else 8)
            kept = 8 if trial % 2 else 4
            for r in range(replicas):
                np.testing.assert_array_equal(sim.history(k, kept, r), ref.history(k, kept, r), err_msg=f"{trial} {r}")
                for a, b in zip(sim.get_state(r)[:2], ref.get_state(r)[:2]):
                    np.testing.assert_array_equal(a, b)
                assert sim.counts(r).tolist() == ref.counts(r).tolist()
        if batched:
            batch.remove(sim)
            batch.close()
        sim.close()
        ref.close()
    c.close(exe)
