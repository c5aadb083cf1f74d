"""The automatic step variant of graphs past the LDS bitmap (2^20 units): the
choice, the same results in every variant, and what a sim whose choice is the
summary still joins and loads as a streaming one."""
import numpy as np
import pytest

import paper_2604_22092_amd as fs
import workloads as W

pytestmark = pytest.mark.gpu

MODEL = {"ei": ("erlang", 3, 1.0), "ir": ("weibull", 2.0, 6.0), "beta": 0.3, "dt": 0.1, "seed": 5}


def _run(sim, steps=12, replicas=1):
    sim.step(steps)
    return [(*sim.get_state(r)[:2], sim.history(0, steps, r)) for r in range(replicas)]


def _seeded(g, n, replicas, **kw):
    sim = fs.Sim.from_model(g, MODEL, replicas=replicas, **kw)
    rng = np.random.default_rng(4)
    st = rng.choice(4, size=n, p=[0.8, 0.05, 0.1, 0.05]).astype(np.int32)
    for r in range(replicas):
        sim.set_state(st, np.zeros(n, np.float32), r, step_index=0)
    return sim


def _same(a, b):
    for x, y in zip(a, b):
        for p, q in zip(x, y):
            np.testing.assert_array_equal(p, q)


CASES = [
    # name, graph, replicas, weighted, chosen variant
    ("er_at_the_limit", lambda: W.erdos_renyi(2**20, 3.0, 1), 1, False, "resident"),
    ("er_past_the_limit", lambda: W.erdos_renyi(2**20 + 1, 3.0, 1), 1, False, "summary"),
    ("ba_two_replicas", lambda: W.barabasi_albert(530_000, 3, 1), 2, False, "summary"),
    ("er_four_replicas", lambda: W.erdos_renyi(270_000, 3.0, 1), 4, False, "stream"),
    ("er_weighted", lambda: W.erdos_renyi(2**20 + 1, 3.0, 1), 1, True, "stream"),
]


@pytest.mark.parametrize("name,graph,replicas,weighted,chosen", CASES, ids=[c[0] for c in CASES])
def test_choice_and_results(name, graph, replicas, weighted, chosen):
    rp, ci = graph()
    n = len(rp) - 1
    w = np.random.default_rng(1).random(len(ci)).astype(np.float32) if weighted else None
    with fs.Graph(rp, ci, w) as g:
        auto = _seeded(g, n, replicas)
        assert auto.variant() == chosen
        got = _run(auto, replicas=replicas)
        auto.close()
        for v in (fs.VARIANT_STREAM, fs.VARIANT_SUMMARY):
            sim = _seeded(g, n, replicas, variant=v)
            _same(got, _run(sim, replicas=replicas))
            sim.close()


def test_an_automatic_summary_joins_a_batch_and_a_chosen_one_does_not():
    rp, ci = W.erdos_renyi(2**20 + 1, 3.0, 1)
    n = len(rp) - 1
    with fs.Graph(rp, ci) as g:
        alone = _seeded(g, n, 1)
        ref = _run(alone)
        alone.close()
        sim = _seeded(g, n, 1)
        chosen = _seeded(g, n, 1, variant=fs.VARIANT_SUMMARY)
        with fs.Batch() as b:
            with pytest.raises(fs.FsError):
                b.add(chosen)
            b.add(sim)
            b.step(12)
            got = [(*sim.get_state(0)[:2], sim.history(0, 12, 0))]
            b.remove(sim)
        _same(ref, got)
        assert sim.variant() == "stream"
        sim.step(5)
        chosen.step(17)
        np.testing.assert_array_equal(sim.get_state(0)[0], chosen.get_state(0)[0])
        sim.close()
        chosen.close()


def test_a_saved_streaming_choice_is_taken(tmp_path):
    rp, ci = W.barabasi_albert(1_060_000, 3, 2)
    n = len(rp) - 1
    path = str(tmp_path / "tuned")
    with fs.Graph(rp, ci) as g:
        sim = _seeded(g, n, 1, variant=fs.VARIANT_STREAM)
        first = sim.autotune(4, variants=False, cache_path=path)
        sim.close()
        sim = _seeded(g, n, 1)
        again = sim.autotune(4, variants=False, cache_path=path)
        assert again["from_cache"] and again["variant"] == first["variant"]
        assert again["heavy_degree"] == first["heavy_degree"]
        got = _run(sim)
        sim.close()
        ref = _seeded(g, n, 1)
        _same(got, _run(ref))
        ref.close()
