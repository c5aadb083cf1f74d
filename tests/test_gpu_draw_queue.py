"""The general step's draw queues against the FP64 oracle.

Units with a positive rate are queued per wavefront and drawn 64 at a time,
what is left after the wavefront's last chunk at once.  The cases load states
that queue anything from none to all 64 units of a chunk, with ages the hazard
table holds and ages it does not, and sit around the sizes where the launch
changes: one partial chunk, one chunk and one more than one chunk per
wavefront for 64 to 1024 threads per workgroup, wavefronts of one to several
chunks, more infections than a push queue holds.  Two steps from each load:
the second reads the ages and infectivity words the first wrote.
"""
import numpy as np
import pytest

import oracle
import paper_2604_22092_amd as fs
import workloads as W
from _parity import check_mismatch_budget, check_one_step

pytestmark = pytest.mark.gpu

EW = {"ei": ("erlang", 3, 1.0), "ir": ("weibull", 2.0, 6.0)}
MIXED, DENSE, SPARSE = [0.5, 0.2, 0.2, 0.1], [0.02, 0.49, 0.49, 0.0], [0.97, 0.01, 0.01, 0.01]

CASES = [
    # name, graph, shares of S E I R, options
    ("one_partial_chunk", lambda: W.random_regular(40, 4, 1), MIXED, {}),
    ("chunks256", lambda: W.random_regular(256 * 64, 6, 1), MIXED, {}),
    ("chunks257", lambda: W.random_regular(256 * 64 + 2, 6, 1), DENSE, {"storage": 1}),
    ("chunks1025", lambda: W.erdos_renyi(1024 * 64 + 1, 6.0, 1), MIXED, {}),
    ("chunks4097", lambda: W.random_regular(4096 * 64 + 2, 5, 1), SPARSE, {"storage": 1}),
    ("chunks4097_full", lambda: W.random_regular(4096 * 64 + 2, 5, 1), DENSE, {}),
    ("passes3_mixed", lambda: W.erdos_renyi(600_001, 4.0, 2), MIXED, {"record_rates": True}),
    ("passes2_bins", lambda: W.barabasi_albert(400_000, 4, 2), MIXED, {"heavy_degree": 16}),
    ("summary", lambda: W.random_regular(600_000, 5, 1), MIXED, {"variant": 3}),
    ("stream", lambda: W.barabasi_albert(300_000, 4, 2), DENSE, {"variant": 1, "storage": 1}),
    ("compaction", lambda: W.erdos_renyi(300_001, 4.0, 2), MIXED, {"compaction": True}),
    ("replicas2", lambda: W.erdos_renyi(150_001, 4.0, 2), MIXED, {"replicas": 2}),
    ("replicas64", lambda: W.random_regular(3000, 6, 2), DENSE, {"replicas": 64, "variant": 2}),
    ("weighted4", lambda: W.erdos_renyi(40_001, 6.0, 2), MIXED, {"replicas": 4, "weighted": True}),
]


@pytest.mark.parametrize("name,graph,shares,opts", CASES, ids=[c[0] for c in CASES])
def test_queued_draws_match_the_oracle(name, graph, shares, opts):
    opts = dict(opts)
    rp, ci = graph()
    n = len(rp) - 1
    rng = np.random.default_rng(8)
    w = rng.random(len(ci)).astype(np.float32) if opts.pop("weighted", False) else None
    gtuple = (rp, ci) if w is None else (rp, ci, w)
    compact = opts.get("storage", 0) == 1
    replicas = opts.get("replicas", 1)
    model = dict(EW, beta=0.3, dt=0.1, seed=2**34 + 3)
    mism = 0
    checked = sorted({0, replicas - 1})
    with fs.Graph(rp, ci, w) as g:
        sim = fs.Sim.from_model(g, model, steps_per_graph=2, **opts)
        for r in range(replicas):
            st = rng.choice(4, size=n, p=shares).astype(np.int32)
            st[: n // 8] = 0          # chunks that queue few units or none
            if compact:
                age = rng.integers(0, 9000, n).astype(np.uint16)
            else:
                age = (rng.random(n) * 12.0).astype(np.float32)
                age[rng.random(n) < 0.5] = np.float32(0.1)  # the age after one step: a table entry
            sim.set_state(st, age, r, step_index=5)
        before = {r: sim.get_state(r)[:2] for r in checked}
        for k in (5, 6):
            sim.step(1)
            for r in checked:
                st, age = before[r]
                ora = oracle.step(gtuple, model, st, age, (st == 2).astype(np.float64), k, replica=r, compact=compact)
                gst, gage, _ = sim.get_state(r)
                got = {"state": gst, "age": gage, "rates": sim.rates(r) if opts.get("record_rates") else None}
                nm, _ = check_one_step(got, ora, st, f"{name} replica {r} step {k}")
                mism += nm
                np.testing.assert_array_equal(sim.history(k, 1, r)[0], np.bincount(gst, minlength=4))
                before[r] = (gst, gage)
        sim.close()
    check_mismatch_budget(mism, 2 * n * len(checked), name)
