"""The replica step (several replicas of a unit-weight graph) against the
general step and the FP64 oracle.

Sims of at least 8192 chunks of 64 units take it; one that records its rates
takes the general kernel, so the two run side by side from the same states.
States, ages and counts must be identical (integer pressures, the same FP32
rates, the same draws).  The cases run groups of 4 and of 8 chunks, on both sides
of the size where 8 take over (3072 of them), their remainders, rows of mixed,
odd, zero and the largest counted degree, and binned rows; groups of 16 are
tested in a file of their own.
"""
import numpy as np
import pytest

import oracle
import paper_2604_22092_amd as fs
import workloads as W

pytestmark = pytest.mark.gpu

EW = {"ei": ("erlang", 3, 1.0), "ir": ("weibull", 2.0, 6.0)}
LN = {"ei": W.LN_E, "ir": W.LN_I}


def _directed(n, degrees, seed):
    """Rows of the given degrees with uniform sources (with multiplicity)."""
    rng = np.random.default_rng(seed)
    rp = np.concatenate([[0], np.cumsum(degrees)]).astype(np.int32)
    return rp, rng.integers(0, n, int(rp[-1])).astype(np.int32)


def _bumpy(n):
    # most rows of 0..9 edges, some of up to 127, so that groups mix degrees
    rng = np.random.default_rng(3)
    d = rng.integers(0, 10, n)
    d[rng.integers(0, n, n // 50)] = rng.integers(10, 128, n // 50)
    d[:3] = 127
    return _directed(n, d, 4)


CASES = [
    # name, graph, replicas, storage, laws, heavy_degree
    ("uniform10_r64", lambda: W.random_regular(8194, 10, 1), 64, 0, LN, 0),
    ("uniform13_r32", lambda: _directed(16_401, np.full(16_401, 13), 2), 32, 1, EW, 0),
    ("uniform3_r8", lambda: _directed(65_601, np.full(65_601, 3), 5), 8, 0, EW, 0),
    ("er10_r16", lambda: W.erdos_renyi(33_001, 10.0, 3), 16, 0, LN, 0),
    ("er10_r16_wide", lambda: W.erdos_renyi(200_003, 10.0, 3), 16, 1, EW, 0),
    ("er6_r4", lambda: W.erdos_renyi(140_001, 6.0, 4), 4, 1, LN, 0),
    ("er6_r8_wide", lambda: W.erdos_renyi(197_001, 6.0, 4), 8, 0, EW, 0),
    ("ba6_r16_hubs", lambda: W.barabasi_albert(40_000, 6, 5), 16, 0, EW, 0),
    ("ba6_r4_hubs_fine", lambda: W.barabasi_albert(140_000, 6, 5), 4, 1, EW, 8),
    ("mixed127_r64", lambda: _bumpy(8_200), 64, 1, LN, 127),
    ("mixed127_r16", lambda: _bumpy(33_000), 16, 0, EW, 127),
]


def _arbitrary(n, compact, seed):
    """A state load's compartments and ages, most of them no fixed step reaches."""
    rng = np.random.default_rng(seed)
    st = rng.choice(4, size=n, p=[0.6, 0.12, 0.12, 0.16]).astype(np.int32)
    if compact:
        return st, rng.integers(0, 9000, n).astype(np.uint16)
    age = (rng.random(n) * 12.0).astype(np.float32)
    age[rng.random(n) < 0.2] = np.float32(0.1)  # the age after one step: a table entry
    return st, age


@pytest.mark.parametrize("name,graph,replicas,storage,laws,hd", CASES, ids=[c[0] for c in CASES])
def test_replica_step_equals_the_general_step(name, graph, replicas, storage, laws, hd):
    rp, ci = graph()
    n = len(rp) - 1
    model = dict(laws, beta=0.08, dt=0.1, seed=2**33 + 5)
    seeds = W.seed_nodes(n, max(20, n // 200), 6)
    loaded = _arbitrary(n, storage == 1, 7)
    outs = []
    with fs.Graph(rp, ci) as g:
        for plain in (True, False):
            sim = fs.Sim.from_model(g, model, replicas=replicas, storage=storage, heavy_degree=hd,
                                    steps_per_graph=8, record_rates=plain)
            sim.seed(seeds, replica=-1)
            # one replica gets a state of its own in the middle of the run: the
            # counts go on from the loaded states, and its ages are evaluated
            sim.step(19)
            sim.set_state(*loaded, replica=replicas - 2)
            sim.step(21)
            outs.append([(*sim.get_state(r)[:2], sim.history(0, 40, r)) for r in range(replicas)])
            sim.close()
    for r, (a, b) in enumerate(zip(*outs)):
        for what, x, y in zip(("states", "ages", "counts"), a, b):
            np.testing.assert_array_equal(x, y, err_msg=f"{name} replica {r}: {what}")
    for r in (0, replicas - 1):
        ost, oage, ohist = oracle.run((rp, ci), model, W.initial_state(n, seeds),
                                      np.zeros(n, np.uint16 if storage == 1 else np.float32), 40, replica=r,
                                      compact=storage == 1)
        np.testing.assert_array_equal(outs[1][r][2], ohist)
        np.testing.assert_array_equal(outs[1][r][0], ost)
        np.testing.assert_array_equal(outs[1][r][1], oage)


def test_replica_step_in_a_batch():
    """Members of several group widths beside one of the general step."""
    specs = [(W.random_regular(8194, 10, 1), 64), (W.erdos_renyi(66_003, 8.0, 2), 16),
             (W.erdos_renyi(200_003, 4.0, 3), 16), (W.random_regular(3000, 8, 4), 4)]
    model = dict(EW, beta=0.08, dt=0.1, seed=9)
    graphs = [fs.Graph(*s) for s, _ in specs]

    def make(i, variant):
        n = len(specs[i][0][0]) - 1
        sim = fs.Sim.from_model(graphs[i], model, replicas=specs[i][1], variant=variant)
        sim.seed(W.seed_nodes(n, n // 100, 5), replica=-1)
        return sim

    alone = []
    for i in range(len(specs)):
        sim = make(i, fs.VARIANT_AUTO)
        sim.step(30)
        alone.append([(*sim.get_state(r)[:2], sim.history(0, 30, r)) for r in (0, specs[i][1] - 1)])
        sim.close()
    members = [make(i, fs.VARIANT_STREAM) for i in range(len(specs))]
    with fs.Batch() as b:
        for m in members:
            b.add(m)
        b.step(11)
        b.step(19)
        for i, m in enumerate(members):
            got = [(*m.get_state(r)[:2], m.history(0, 30, r)) for r in (0, specs[i][1] - 1)]
            for x, y in zip(alone[i], got):
                for p, q in zip(x, y):
                    np.testing.assert_array_equal(p, q, err_msg=f"member {i}")
        for m in members:
            b.remove(m)
    for m in members:
        m.close()
    for g in graphs:
        g.close()


def test_replica_step_left_and_entered_by_new_bins():
    """Bins whose light rows pass the counted degrees run the general step."""
    rp, ci = W.barabasi_albert(40_000, 6, 5)
    model = dict(EW, beta=0.08, dt=0.1, seed=9)
    ref = None
    with fs.Graph(rp, ci) as g:
        for bins in ([0, 0, 0], [0, -1, 12], [-1, 200, 0]):
            sim = fs.Sim.from_model(g, model, replicas=16, variant=fs.VARIANT_SUMMARY)
            sim.seed(W.seed_nodes(40_000, 200, 5), replica=-1)
            for hd in bins:
                sim.set_bins(hd)
                sim.step(12)
            got = [(*sim.get_state(r)[:2], sim.history(0, 36, r)) for r in range(16)]
            sim.close()
            ref = ref or got
            for x, y in zip(ref, got):
                for p, q in zip(x, y):
                    np.testing.assert_array_equal(p, q, err_msg=str(bins))


def test_replica_step_counts_over_a_short_ring():
    """A launch sequence longer than the count ring keeps the last rows."""
    rp, ci = W.random_regular(8200, 6, 3)
    model = dict(LN, beta=0.2, dt=0.1, seed=4)
    rows = []
    with fs.Graph(rp, ci) as g:
        for ring, spg in ((0, 0), (5, 0), (7, 40)):
            sim = fs.Sim.from_model(g, model, replicas=64, history_len=ring, steps_per_graph=spg)
            sim.seed(W.seed_nodes(8200, 50, 1), replica=-1)
            sim.step(80)
            rows.append(sim.history(75, 5, 63))
            sim.close()
    np.testing.assert_array_equal(rows[0], rows[1])
    np.testing.assert_array_equal(rows[0], rows[2])
    assert np.all(rows[0].sum(1) == 8200)
