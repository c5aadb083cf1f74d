"""The replica step with groups of 16 chunks, which takes REPS_GROUPS16 of them:
at that many and just above, for 16, 32 and 64 replicas, both storages, uniform
and mixed rows, binned rows, a partial last group, and in a batch, against the
general step (rates recorded) and the FP64 oracle."""
import os
import re

import numpy as np
import pytest

import oracle
import paper_2604_22092_amd as fs
import workloads as W
from test_gpu_replica_step import EW, LN, _arbitrary, _bumpy, _directed

pytestmark = pytest.mark.gpu

CSRC = os.path.join(os.path.dirname(os.path.abspath(fs.__file__)), "csrc")


def _constant(name):
    text = open(os.path.join(CSRC, "fs_internal.hpp")).read()
    return int(re.search(rf"constexpr \w+ {name} = (\d+);", text).group(1))


CHUNKS = 16 * _constant("REPS_GROUPS16")  # the fewest 64-unit chunks in groups of 16


def _nodes(replicas):
    return CHUNKS * 64 // replicas


CASES = [
    # name, nodes past the fewest, graph, replicas, storage, laws, heavy_degree
    ("uniform6_r16", 0, lambda n: W.random_regular_matchings(n, 6, 1), 16, 0, LN, 0),
    ("uniform13_r64_partial", 3, lambda n: _directed(n, np.full(n, 13), 2), 64, 1, EW, 0),
    ("er8_r16_partial", 37, lambda n: W.erdos_renyi(n, 8.0, 3), 16, 0, EW, 0),
    ("er8_r32_compact", 1, lambda n: W.erdos_renyi(n, 8.0, 3), 32, 1, LN, 0),
    ("ba5_r16_hubs", 17, lambda n: W.barabasi_albert(n, 5, 5), 16, 1, EW, 12),
    ("ba5_r32_hubs", 0, lambda n: W.barabasi_albert(n, 5, 5), 32, 0, EW, 0),
    ("mixed127_r64", 9, _bumpy, 64, 0, LN, 127),
]


@pytest.mark.parametrize("name,more,graph,replicas,storage,laws,hd", CASES, ids=[c[0] for c in CASES])
def test_groups_of_16_equal_the_general_step(name, more, graph, replicas, storage, laws, hd):
    n = _nodes(replicas) + more
    rp, ci = graph(n)
    assert len(rp) == n + 1 and (n * replicas + 63) // 64 >= CHUNKS
    model = dict(laws, beta=0.08, dt=0.1, seed=2**33 + 5)
    seeds = W.seed_nodes(n, n // 100, 6)
    loaded = _arbitrary(n, storage == 1, 7)
    some = sorted({0, 1, replicas // 2, replicas - 2, replicas - 1})
    outs = []
    with fs.Graph(rp, ci) as g:
        for plain in (True, False):
            sim = fs.Sim.from_model(g, model, replicas=replicas, storage=storage, heavy_degree=hd, steps_per_graph=6,
                                    record_rates=plain)
            sim.seed(seeds, replica=-1)
            sim.step(7)
            sim.set_state(*loaded, replica=replicas - 2)
            sim.step(9)
            outs.append([(*sim.get_state(r)[:2], sim.history(0, 16, r)) for r in some])
            sim.close()
    for r, a, b in zip(some, *outs):
        for what, x, y in zip(("states", "ages", "counts"), a, b):
            np.testing.assert_array_equal(x, y, err_msg=f"{name} replica {r}: {what}")
    want = oracle.run((rp, ci), model, W.initial_state(n, seeds), np.zeros(n, np.uint16 if storage else np.float32), 16,
                      replica=replicas - 1, compact=storage == 1)
    for x, y in zip(outs[1][-1], want):
        np.testing.assert_array_equal(x, y)


def test_groups_of_16_in_a_batch():
    """Beside members of narrower groups and one of the general step."""
    model = dict(EW, beta=0.08, dt=0.1, seed=9)
    specs = [(W.erdos_renyi(3000, 8.0, 4), 4), (W.barabasi_albert(_nodes(16) + 5, 4, 3), 16),
             (W.random_regular(8194, 10, 1), 64), (W.erdos_renyi(_nodes(32), 6.0, 2), 32)]
    graphs = [fs.Graph(*s) for s, _ in specs]

    def make(i):
        n = len(specs[i][0][0]) - 1
        sim = fs.Sim.from_model(graphs[i], model, replicas=specs[i][1], variant=fs.VARIANT_STREAM)
        sim.seed(W.seed_nodes(n, n // 100, 5), replica=-1)
        return sim

    def read(i, sim):
        return [(*sim.get_state(r)[:2], sim.history(0, 20, r)) for r in (0, specs[i][1] - 1)]

    alone = []
    for i in range(len(specs)):
        sim = make(i)
        sim.step(20)
        alone.append(read(i, sim))
        sim.close()
    members = [make(i) for i in range(len(specs))]
    with fs.Batch() as b:
        for m in members:
            b.add(m)
        b.step(7)
        b.step(13)
        for i, m in enumerate(members):
            for x, y in zip(alone[i], read(i, m)):
                for p, q in zip(x, y):
                    np.testing.assert_array_equal(p, q, err_msg=f"member {i}")
        for m in members:
            b.remove(m)
    for m in members:
        m.close()
    for g in graphs:
        g.close()
