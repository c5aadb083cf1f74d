"""Timed cases of the renewal tau-leap framework.

Each case is one unit of work a program hands to the framework through its
public entry points, at the sizes the named workloads, the benchmark and the
serving mix of this repository use, from the smallest calls (where launches
and latency count) to ones that fill the card:

  solve      a trajectory of one sim that the program keeps (its step loop is
             captured): load the initial state, run the steps, read the
             per-step counts and the final state
  ensemble   a scenario solve on a resident graph: create the sim, seed it, run
             the steps, read every replica's counts (and, where "states" is
             set, every replica's final state), release the sim
  nowcast    one recorded step from an observed state: load it, step once, read
             the rates and the state (the inspection and checkpoint path)
  markov     a trajectory of the Markovian engine
  server     a burst of scenario requests to the continuous-batching server

Graphs are seeded random ones of the paper's families (fixed degree,
Erdos-Renyi, Barabasi-Albert), generated on the GPU.
"""
import math

import numpy as np
import torch

import paper_2604_22092_amd as fs

LN = "ln"          # E ~ LN(ln 3, 0.5), I ~ LN(ln 5, 0.6)
EW = "ew"          # E ~ Erlang(3, rate 1), I ~ Weibull(2, 6)
WE = "we"          # E ~ Weibull(2, 4), I ~ Erlang(4, mean 5)
PAPER = "paper"    # the paper's default: E mean 5 d / median 4 d, I mean 7.5 d / median 5 d
LAWS = {
    LN: (("lognormal", math.log(3.0), 0.5), ("lognormal", math.log(5.0), 0.6)),
    EW: (("erlang", 3, 1.0), ("weibull", 2.0, 6.0)),
    WE: (("weibull", 2.0, 4.0), ("erlang", 4, 0.8)),
    PAPER: (("lognormal", math.log(4.0), math.sqrt(2.0 * math.log(5.0 / 4.0))),
            ("lognormal", math.log(5.0), math.sqrt(2.0 * math.log(7.5 / 5.0)))),
}
SHED_LAW = ("lognormal", math.log(2.5), 0.5)   # viral-load curve, median 2.5 d
SHED_SCALE = 5.0


def _sim(kind, **kw):
    c = {"kind": kind, "graph": "regular", "n": 10_000, "deg": 10, "laws": LN, "beta": 0.06, "dt": 0.1,
         "steps": 300, "seeds": 10, "replicas": 1, "compact": False, "weighted": False, "shed": "none",
         "adaptive": False, "compaction": False, "heavy_degree": 0, "steps_per_graph": 50, "states": True}
    c.update(kw)
    return c


def listed():
    return [
        # the small parity workload: a step is launches and latency, no bandwidth
        _sim("solve", name="regular10_n1e4"),
        # the flagship: random 10-regular, captured loop, one replica, FP32
        _sim("solve", name="regular10_n1e6", n=1_000_000, steps=500, seeds=100),
        # heavy-tailed degrees, the autotuner's usual bins
        _sim("solve", name="ba5_n1e6", graph="ba", n=1_000_000, deg=5, laws=EW, beta=0.03, steps=500, seeds=100,
             heavy_degree=12),
        # adaptive step size on the paper's own default workload
        _sim("solve", name="adaptive_er8_n1e6", graph="er", n=1_000_000, deg=8, laws=PAPER, beta=0.25, steps=300,
             seeds=100, adaptive=True),
        # a national-scale graph in compact storage: more nodes than the LDS holds bits for
        _sim("ensemble", name="regular8_n1e7_compact", n=10_000_000, deg=8, beta=0.07, dt=0.2, steps=200, seeds=1000,
             compact=True, steps_per_graph=0),
        # a scenario of the serving mix solved alone: 16 replicas on a heavy-tailed graph
        _sim("ensemble", name="ba4_n3e5_r16", graph="ba", n=300_000, deg=4, laws=WE, beta=0.05, seeds=300,
             replicas=16, steps_per_graph=0, states=False),
        # many replicas of a town-sized graph, compact storage, states kept
        _sim("ensemble", name="regular6_n2e4_r64", n=20_000, deg=6, beta=0.08, seeds=20, replicas=64, compact=True,
             steps_per_graph=0),
        # a weighted contact graph, a few replicas
        _sim("ensemble", name="weighted_er10_n2e5_r4", graph="er", n=200_003, deg=10, laws=EW, beta=0.06, steps=200,
             seeds=200, replicas=4, weighted=True, steps_per_graph=0),
        # age-dependent infectiousness on an odd-sized graph
        _sim("ensemble", name="shed_regular10_n3e5", n=300_001, deg=10, laws=LN, beta=0.06, seeds=300, shed="density",
             steps_per_graph=0),
        # rates of one step from an observed state (weighted, age-dependent shedding, hubs)
        _sim("nowcast", name="nowcast_ba6_n1e5", graph="ba", n=100_003, deg=6, steps=1, shed="density", weighted=True,
             steps_per_graph=0),
        # the Markovian engine over a whole SIR epidemic
        {"name": "markov_er8_n1e6", "kind": "markov", "graph": "er", "n": 1_000_000, "deg": 8, "model": "sir",
         "beta": 0.25, "sigma": 0.3, "gamma": 0.15, "steps": 600, "seeds": 100, "steps_per_graph": 50},
        # continuous batching: a burst of requests of uneven size over a pool of resident graphs
        {"name": "server_burst24", "kind": "server", "requests": 24, "pool": 6, "n_min": 10_000, "n_max": 200_000,
         "replicas": 16, "steps": 300, "compact": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "ensemble", "ensemble", "ensemble", "nowcast", "markov", "server"])
    graph = rng.choice(["regular", "er", "ba"])
    deg = rng.randint(2, 8) if graph == "ba" else rng.randint(4, 16)
    laws = rng.choice([LN, EW, WE])
    beta = round(rng.uniform(0.02, 0.1), 4)
    steps = rng.randint(100, 400)
    if kind == "server":
        return {"kind": "server", "requests": rng.randint(4, 24), "pool": rng.randint(2, 6), "n_min": 10_000,
                "n_max": _log(rng, 20_000, 200_000), "replicas": 16, "steps": rng.randint(100, 300),
                "compact": rng.random() < 0.3}
    if kind == "markov":
        return {"kind": "markov", "graph": graph, "n": _log(rng, 1e4, 1e6), "deg": deg,
                "model": rng.choice(["sir", "seir", "sis"]), "beta": round(rng.uniform(0.1, 0.3), 4), "sigma": 0.3,
                "gamma": 0.15, "steps": steps, "seeds": 100, "steps_per_graph": rng.choice([0, 25, 50])}
    if kind == "nowcast":
        return _sim("nowcast", graph=graph, n=_log(rng, 1e4, 3e5), deg=deg, laws=laws, beta=beta, steps=1,
                    shed=rng.choice(["none", "density"]), weighted=rng.random() < 0.5, steps_per_graph=0)
    if kind == "solve":
        n = _log(rng, 1e4, 1.5e6)
        adaptive = rng.random() < 0.25
        return _sim("solve", graph=graph, n=n, deg=deg, laws=laws, beta=beta, steps=steps, seeds=max(10, n // 5000),
                    compact=not adaptive and rng.random() < 0.4, adaptive=adaptive,
                    heavy_degree=rng.choice([0, 12, 32]), compaction=not adaptive and rng.random() < 0.15,
                    steps_per_graph=rng.choice([0, 20, 50]))
    replicas = rng.choice([1, 2, 4, 8, 16, 16, 32, 64])
    n = _log(rng, 1e4, min(3e6, 5e6 / replicas))
    weighted = rng.random() < 0.25
    shed = "density" if not weighted and replicas <= 4 and rng.random() < 0.3 else "none"
    return _sim("ensemble", graph=graph, n=n, deg=deg, laws=laws, beta=beta, steps=steps, seeds=max(10, n // 1000),
                replicas=replicas, compact=rng.random() < 0.4, weighted=weighted, shed=shed, steps_per_graph=0,
                states=n * replicas <= 1_500_000)


# ------------------------------------------------------------------- graphs

def _csr(n, rows, cols):
    key = torch.sort(rows * n + cols).values
    ptr = torch.zeros(n + 1, dtype=torch.int64, device=key.device)
    ptr[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0)
    return ptr.to(torch.int32).cpu().numpy(), (key % n).to(torch.int32).cpu().numpy()


def _both(n, a, b):
    return _csr(n, torch.cat([a, b]), torch.cat([b, a]))


def _graph(family, n, deg, g, dev):
    """Incoming CSR of a symmetric random graph (int32 host arrays)."""
    if family == "regular":
        # random Hamiltonian cycles, and for an odd degree a random matching
        part = []
        for _ in range(deg // 2):
            p = torch.randperm(n, generator=g, device=dev)
            for shift in (1, -1):
                q = torch.empty(n, dtype=torch.int32, device=dev)
                q[p] = torch.roll(p, shift).to(torch.int32)
                part.append(q)
        if deg % 2:
            p = torch.randperm(n, generator=g, device=dev)
            q = torch.empty(n, dtype=torch.int32, device=dev)
            q[p] = p.view(-1, 2).flip(1).reshape(-1).to(torch.int32)
            part.append(q)
        col = torch.sort(torch.stack(part, 1), dim=1).values
        return np.arange(0, n * deg + 1, deg, dtype=np.int32), col.reshape(-1).cpu().numpy()
    if family == "er":
        m = n * deg // 2
        a = torch.randint(0, n, (m,), generator=g, device=dev)
        b = (a + torch.randint(1, n, (m,), generator=g, device=dev)) % n
        return _both(n, a, b)
    # Barabasi-Albert: every far endpoint is a uniform pick of the endpoints placed before it
    # (the picks of odd slots are followed until they name a node), from K_{m+1}
    m = deg
    cu, cv = torch.triu_indices(m + 1, m + 1, 1, device=dev)
    clique = torch.stack([cu, cv], 1).reshape(-1)
    base = clique.numel()
    j = torch.arange((n - m - 1) * m, device=dev)
    owner = (m + 1) + j // m
    bound = base + 2 * j + 1
    r = torch.minimum((torch.rand(j.numel(), generator=g, device=dev, dtype=torch.float64) * bound).long(), bound - 1)
    p = r.clone()
    while True:
        odd = (p >= base) & ((p - base) % 2 == 1)
        if not bool(odd.any()):
            break
        p = torch.where(odd, r[((p - base - 1) // 2).clamp(min=0)], p)
    far = torch.where(p < base, clique[p.clamp(max=base - 1)], (m + 1) + ((p - base) // 2) // m)
    src, dst = torch.cat([cu, owner]), torch.cat([cv, far])
    key = torch.unique(torch.minimum(src, dst) * n + torch.maximum(src, dst))
    a, b = key // n, key % n
    return _both(n, a[a != b], b[a != b])


class _Held:
    """What the program keeps between calls; handles are released with it."""

    def __init__(self, case):
        self.case = case
        self.held = []

    def keep(self, x):
        self.held.append(x)
        return x

    def __del__(self):
        for x in reversed(self.held):
            try:
                x.close()
            except Exception:
                pass


def _pick(rng, n, count):
    return np.sort(rng.choice(n, size=min(count, n), replace=False)).astype(np.int64)


def _even(n, family, deg):
    return n + (n & 1) if family == "regular" and deg % 2 else n


def _weights(rng, nnz):
    return rng.lognormal(-0.1, 0.45, nnz).astype(np.float32)


def _observed(rng, n, dt):
    """An observed mid-epidemic state: compartments and ages of a fixed-step run."""
    state = rng.choice(4, size=n, p=[0.55, 0.1, 0.15, 0.2]).astype(np.int32)
    ages = np.concatenate([[np.float32(0)], np.cumsum(np.full(160, dt, np.float32), dtype=np.float32)])
    return state, ages[rng.integers(0, 161, n)].astype(np.float32)


def _sim_kw(c):
    return {"replicas": c["replicas"], "storage": fs.FS_STORAGE_COMPACT if c["compact"] else fs.FS_STORAGE_FP32,
            "steps_per_graph": c["steps_per_graph"], "heavy_degree": c["heavy_degree"], "adaptive": c["adaptive"],
            "compaction": c["compaction"], "record_rates": c["kind"] == "nowcast"}


def _model(c, seed):
    ei, ir = LAWS[c["laws"]]
    return {"ei": ei, "ir": ir, "beta": c["beta"], "dt": c["dt"], "seed": seed,
            "shed": ("density", SHED_LAW, SHED_SCALE) if c["shed"] == "density" else None}


def _inputs(case, seed):
    """Graph arrays, edge weights and the host generator of a case."""
    dev = torch.device("cuda", 0)
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    rng = np.random.default_rng(seed)
    n = _even(case["n"], case["graph"], case["deg"])
    rp, ci = _graph(case["graph"], n, case["deg"], g, dev)
    w = _weights(rng, len(ci)) if case.get("weighted") else None
    return n, rp, ci, w, rng


def prepare(case, seed):
    s = _Held(case)
    if case["kind"] == "server":
        dev = torch.device("cuda", 0)
        g = torch.Generator(device=dev)
        g.manual_seed(seed)
        rng = np.random.default_rng(seed)
        sizes, s.graphs, s.requests = [], [], []
        for i in range(case["pool"]):
            fam = ("regular", "er", "ba")[i % 3]
            deg = int(rng.integers(2, 9) if fam == "ba" else rng.integers(4, 17) if fam == "regular" else 10)
            # sizes spread evenly (in log) over the range, smallest and largest included
            n = case["n_min"] * (case["n_max"] / case["n_min"]) ** (i / max(1, case["pool"] - 1))
            n = _even(int(round(n)), fam, deg)
            sizes.append(n)
            s.graphs.append(s.keep(fs.Graph(*_graph(fam, n, deg, g, dev))))
        for i in range(case["requests"]):
            gi = i % case["pool"]
            ei, ir = LAWS[(LN, EW, WE)[int(rng.integers(0, 3))]]
            s.requests.append((gi, ei, ir, float(rng.uniform(0.02, 0.1)), 0.1, int(rng.integers(0, 2**62)),
                               _pick(rng, sizes[gi], max(10, sizes[gi] // 1000))))
        s.server = s.keep(fs.Server(storage=fs.FS_STORAGE_COMPACT if case["compact"] else fs.FS_STORAGE_FP32))
        return s
    n, rp, ci, w, rng = _inputs(case, seed)
    s.n = n
    s.graph = s.keep(fs.Graph(rp, ci, w))
    if case["kind"] == "markov":
        s.engine = s.keep(fs.Markov(s.graph, {"model": case["model"], "beta": case["beta"], "sigma": case["sigma"],
                                              "gamma": case["gamma"], "theta": 0.01, "p_max": 0.1, "tau_max": 1.0,
                                              "seed": seed}, steps_per_graph=case["steps_per_graph"]))
        s.state0 = np.zeros(n, np.int32)
        s.state0[_pick(rng, n, case["seeds"])] = 2
        return s
    s.model = _model(case, seed)
    if case["kind"] == "nowcast":
        s.state0, s.age0 = _observed(rng, n, case["dt"])
    else:
        s.nodes = _pick(rng, n, case["seeds"])
        s.state0 = np.zeros(n, np.int32)
        s.state0[s.nodes] = 1
        s.age0 = np.zeros(n, np.uint16 if case["compact"] else np.float32)
    if case["kind"] != "ensemble":
        s.sim = s.keep(fs.Sim.from_model(s.graph, s.model, **_sim_kw(case)))
    return s


def _states(sim):
    return [sim.get_state(r)[:2] for r in range(sim.replicas)]


def run(s):
    c = s.case
    k = c["steps"]
    if c["kind"] == "server":
        ids = [s.server.submit(s.graphs[gi], ei, ir, beta, dt, seed, c["replicas"], k, nodes)
               for gi, ei, ir, beta, dt, seed, nodes in s.requests]
        out = []
        for i in ids:
            s.server.wait(i)
            out.append(s.server.result(i)[0])
        return out
    if c["kind"] == "markov":
        s.engine.set_state(s.state0, step_index=0)
        s.engine.step(k)
        counts, taus, events = s.engine.history(0, k)
        return {"counts": counts, "taus": taus, "events": events, "state": s.engine.get_state()[0]}
    if c["kind"] == "ensemble":
        sim = fs.Sim.from_model(s.graph, s.model, **_sim_kw(c))
        sim.seed(s.nodes)
        sim.step(k)
        out = {"history": [sim.history(0, k, r) for r in range(c["replicas"])]}
        if c["states"]:
            st = _states(sim)
            out["state"], out["age"] = np.stack([x[0] for x in st]), np.stack([x[1] for x in st])
        out["history"] = np.stack(out["history"])
        sim.close()
        return out
    sim = s.sim
    sim.set_state(s.state0, s.age0, 0, step_index=0)
    sim.step(k)
    if c["kind"] == "nowcast":
        st, age = sim.get_state()[:2]
        return {"rates": sim.rates(), "state": st, "age": age}
    out = {"history": sim.history(0, k)}
    if c["adaptive"]:
        out["sizes"] = sim.step_sizes(0, k)
    out["state"], out["age"] = sim.get_state()[:2]
    return out


# --------------------------------------------------------------------- work

def _edges(graph, n, deg):
    return n * (2 * deg if graph == "ba" else deg)


def work(case):
    """One step reads every edge's source id (and weight) and every unit's
    infectivity bit once and reads and writes every unit's state and age once;
    one addition per edge and replica, one draw per unit."""
    k = case["steps"]
    if case["kind"] == "server":
        b = f = 0.0
        for i in range(case["requests"]):
            n = case["n_min"] * (case["n_max"] / case["n_min"]) ** ((i % case["pool"]) / max(1, case["pool"] - 1))
            unit = 6 if case["compact"] else 16
            b += k * n * (4 * 10 + case["replicas"] * (unit + 0.25))
            f += k * n * case["replicas"] * (10 + 1)
        return {"bytes": b, "flops": f}
    n, e = case["n"], _edges(case["graph"], case["n"], case["deg"])
    if case["kind"] == "markov":
        # state r/w, influence, and the pushed influences of every node's one change into and out of I
        return {"bytes": k * n * 6.0 + 16.0 * e, "flops": k * n + 2.0 * e}
    r = case["replicas"]
    unit = 6 if case["compact"] else 16
    b = k * (e * (8 if case["weighted"] else 4) + n * r * (unit + 0.25))
    if case["kind"] == "nowcast":
        b += n * 20.0
    return {"bytes": float(b), "flops": float(k * (e * r + n * r))}


# -------------------------------------------------------------------- exact

def _hazard64(law, t):
    """f/S of a holding-time law in 64 bits (0 at age 0 for the log-normal)."""
    if law[0] == "lognormal":
        x = torch.clamp(t, min=1e-300)
        z = (torch.log(x) - law[1]) / (law[2] * math.sqrt(2.0))
        h = math.sqrt(2.0 / math.pi) / (law[2] * x * torch.special.erfcx(z))
        return torch.where(t > 0, h, torch.zeros_like(h))
    if law[0] == "weibull":
        return law[1] / law[2] * (t / law[2]) ** (law[1] - 1.0)
    y = law[2] * t
    term, tot = torch.ones_like(y), torch.ones_like(y)
    for j in range(1, law[1]):
        term = term * y / j
        tot = tot + term
    return law[2] * term / tot


def _shed64(t):
    x = torch.clamp(t, min=1e-300)
    z = (torch.log(x) - SHED_LAW[1]) / SHED_LAW[2]
    f = SHED_SCALE * torch.exp(-0.5 * z * z) / (x * SHED_LAW[2] * math.sqrt(2.0 * math.pi))
    return torch.where(t > 0, f, torch.zeros_like(f))


def _philox(ctr, seed):
    """Word 0 of Philox4x32-10 at counters (node, 0, 0, 0)."""
    x = [ctr.astype(np.uint64)] + [np.zeros(len(ctr), np.uint64) for _ in range(3)]
    k0, k1, mask = seed & 0xFFFFFFFF, seed >> 32, np.uint64(0xFFFFFFFF)
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * x[0], np.uint64(0xCD9E8D57) * x[2]
        x = [(p1 >> np.uint64(32)) ^ x[1] ^ np.uint64(k0), p1 & mask, (p0 >> np.uint64(32)) ^ x[3] ^ np.uint64(k1),
             p0 & mask]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return x[0]


def exact(case, seed):
    """One step's rates and ages in 64 bits.  A trajectory has no 64-bit value
    to be compared unit by unit: one draw decided otherwise changes it all."""
    if case["kind"] != "nowcast":
        return None
    n, rp, ci, w, rng = _inputs(case, seed)
    state, age = _observed(rng, n, case["dt"])
    ei, ir = LAWS[case["laws"]]
    x, t = torch.from_numpy(state), torch.from_numpy(age).double()
    iota = (_shed64(t) if case["shed"] == "density" else torch.ones(n, dtype=torch.float64)) * (x == 2)
    edge = iota[torch.from_numpy(ci).long()]
    if w is not None:
        edge = edge * torch.from_numpy(w).double()
    row = torch.repeat_interleave(torch.arange(n), torch.from_numpy(np.diff(rp)).long())
    p = torch.zeros(n, dtype=torch.float64).index_add_(0, row, edge)
    zero = torch.zeros(n, dtype=torch.float64)
    lam = torch.where(x == 0, case["beta"] * p, zero)
    lam = torch.where(x == 1, _hazard64(ei, t), lam)
    lam = torch.where(x == 2, _hazard64(ir, t), lam)
    u = torch.from_numpy((_philox(np.arange(n), seed) >> np.uint64(8)).astype(np.float64) * 2.0**-24)
    fire = (lam > 0) & (u < -torch.expm1(-lam * case["dt"]))
    return {"rates": lam.numpy(), "state": None, "age": torch.where(fire, zero, t + case["dt"]).numpy()}
