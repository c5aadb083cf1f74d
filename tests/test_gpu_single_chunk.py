"""Uniform layouts whose wavefronts have one 64-unit chunk each draw in place,
larger ones through the queue: both sides of the edge (4096 wavefronts of an
LDS variant on 256 compute units), workgroups of 64 to 1024 threads, ages the
hazard table holds and ones it does not, and shedding, against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2604_22092_amd as fs
import workloads as W

pytestmark = pytest.mark.gpu

EW = {"ei": ("erlang", 3, 1.0), "ir": ("weibull", 2.0, 6.0)}
LN = {"ei": W.LN_E, "ir": W.LN_I}

CASES = [
    # name, nodes, replicas, storage, laws, shedding
    ("one_chunk", 64, 1, 0, LN, None),
    ("waves1", 16_384, 1, 0, EW, None),
    ("waves2_odd", 16_386, 1, 1, LN, None),
    ("waves12_r4", 40_002, 4, 0, EW, None),
    ("waves16_r16", 15_000, 16, 1, LN, None),
    ("last_single_r16", 16_384, 16, 0, EW, None),
    ("first_queued_r16", 16_388, 16, 0, EW, None),
    ("last_single_r1", 262_144, 1, 0, LN, None),
    ("first_queued_r1", 262_146, 1, 1, LN, None),
    ("shed_r1", 100_000, 1, 0, EW, ("density", ("lognormal", 0.9, 0.5), 4.0)),
]


@pytest.mark.parametrize("name,n,replicas,storage,laws,shed", CASES, ids=[c[0] for c in CASES])
def test_draws_in_place_and_queued(name, n, replicas, storage, laws, shed):
    rp, ci = W.random_regular_matchings(n, 6, 3)
    model = dict(laws, beta=0.1, dt=0.1, seed=2**33 + 5, shed=shed)
    compact = storage == 1
    rng = np.random.default_rng(7)
    st = rng.choice(4, size=n, p=[0.6, 0.12, 0.12, 0.16]).astype(np.int32)
    if compact:
        age = rng.integers(0, 9000, n).astype(np.uint16)
    else:
        age = (rng.random(n) * 12.0).astype(np.float32)
        age[rng.random(n) < 0.5] = np.float32(0.1)  # the age after one step: a table entry
    last = replicas - 1
    with fs.Graph(rp, ci) as g:
        sim = fs.Sim.from_model(g, model, replicas=replicas, storage=storage, variant=fs.VARIANT_RESIDENT)
        for r in range(replicas):
            sim.set_state(st, age, r, step_index=0)
        sim.step(12)
        got = (*sim.get_state(last)[:2], sim.history(0, 12, last))
        sim.close()
    want = oracle.run((rp, ci), model, st, age, 12, replica=last, compact=compact)
    for what, a, b in zip(("states", "ages", "counts"), got, want):
        np.testing.assert_array_equal(a, b, err_msg=what)
