"""The autotuner's saved choices and candidates: choices saved by a version
whose step kernels were others are made anew, and bins that leave the replica
step are tried in every variant."""
import numpy as np
import pytest
import torch  # (at collection, before any test loads the library: one HIP runtime for both)

import paper_2604_22092_amd as fs
import workloads as W

pytestmark = pytest.mark.gpu

MODEL = {"ei": ("erlang", 3, 1.0), "ir": ("weibull", 2.0, 6.0), "beta": 0.08, "dt": 0.1, "seed": 9}


def _signature(version, rp, replicas):
    """The tune file's key of a plain FP32 sim (FNV-1a)."""
    deg = np.diff(rp)
    h = 1469598103934665603

    def add(raw):
        nonlocal h
        for b in raw:
            h = ((h ^ b) * 1099511628211) & (2**64 - 1)

    add(version.encode())
    add(np.int32(torch.cuda.get_device_properties(0).multi_processor_count).tobytes())
    add(np.int64(len(deg)).tobytes() + np.int64(rp[-1]).tobytes())
    add(np.array([replicas, 0, 0, 0, 0, 0, 0], np.int32).tobytes())
    for d, c in enumerate(np.bincount(deg)):
        if c:
            add(np.int64(d).tobytes() + np.int64(c).tobytes())
    return f"{h:016x}"


def test_an_older_choice_is_made_anew(tmp_path):
    rp, ci = W.barabasi_albert(140_000, 5, 2)
    path = str(tmp_path / "tuned")
    with open(path, "w") as f:
        f.write(f"{_signature('flashspread-tune-1', rp, 4)} variant=1 heavy_degree=-1 segment_edges=512 "
                "us_per_step=1.0\n")
    with fs.Graph(rp, ci) as g:
        sim = fs.Sim.from_model(g, MODEL, replicas=4)
        res = sim.autotune(3, variants=True, cache_path=path)
        assert res["signature"] == _signature("flashspread-tune-2", rp, 4)
        assert not res["from_cache"] and res["trials"] > 1
        again = fs.Sim.from_model(g, MODEL, replicas=4)
        assert again.autotune(3, variants=True, cache_path=path)["from_cache"]
        sim.close()
        again.close()


def test_bins_that_leave_the_replica_step_are_tried_in_every_variant():
    rp, ci = W.barabasi_albert(140_000, 5, 2)
    top = int(np.diff(rp).max())
    assert top > 256
    bins = [64, -1] + [t for t in (8, 12, 16, 24, 32, 128, 256) if t < top]
    leaving = [b for b in bins if b < 0 or b > 127]
    with fs.Graph(rp, ci) as g:
        sim = fs.Sim.from_model(g, MODEL, replicas=4)
        ref = fs.Sim.from_model(g, MODEL, replicas=4)
        for s in (sim, ref):
            s.seed(np.arange(200), replica=-1)
        res = sim.autotune(3, variants=True)
        # (560000 units: resident, summary and streaming)
        assert res["trials"] == len(bins) + 2 * len(leaving)
        sim.step(20)
        ref.step(20)
        for r in range(4):
            np.testing.assert_array_equal(sim.history(0, 20, r), ref.history(0, 20, r))
            np.testing.assert_array_equal(sim.get_state(r)[0], ref.get_state(r)[0])
        sim.close()
        ref.close()
