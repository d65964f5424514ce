"""The work that users of this engine have it do, as cases that can be timed.

A case is one call of a public entry point, whole: ``Solver.run`` with its
results read back, a ``FusedBatch`` run, or a ``PoolServer`` serving a queue.
``listed()`` holds the fixed cases, ``draw()`` gives more of the same ranges;
both are read by ``prepare`` (inputs, from a seed), ``run`` (one pass) and
``work`` (what the pass cannot do without).

Every output is a whole number (energies, cuts, spins, counts), so two
versions of the engine agree on a case only if they agree bit for bit, and
``exact`` has no rounded value to give.
"""
from __future__ import annotations

import math

import numpy as np

from paper_2510_21105_amd import pa, serve
from paper_2510_21105_amd import workloads as W


def listed() -> list:
    return [
        # The smallest call: a 20-node instance, as in a check against
        # exhaustive search; latency and launches are all there is.
        dict(name="tiny-20", kind="random", n=20, m=60, signed=False, order="natural", R=128, K=50, S=10,
             beta1=3.0, population=True),
        # A first solve of a small benchmark graph, its population read back
        # (sampling, not only the best configuration).
        dict(name="small-800", kind="random", n=800, m=4000, signed=False, order="natural", R=128, K=50, S=10,
             beta1=3.0, population=True),
        # The benchmark's dense family: few nodes, long adjacency rows.
        dict(name="rows48-800", kind="random", n=800, m=19200, signed=False, order="natural", R=1024, K=50, S=10,
             beta1=3.0),
        # Degrees above 127, which only the word kernel takes.
        dict(name="rows200-1000", kind="random", n=1000, m=100000, signed=False, order="natural", R=1024, K=20,
             S=5, beta1=1.0, population=True),
        # Signed weights on a mid-sized random graph, noise levels and pair
        # cluster moves on.
        dict(name="signed-2000", kind="random", n=2000, m=20000, signed=True, order="natural", R=2048, K=100,
             S=10, beta1=4.0, as_enable=1, nl_period=10),
        # A ragged population on a sparse graph, temperature steps chosen by
        # the run itself.
        dict(name="adaptive-3001", kind="random", n=3001, m=9001, signed=False, order="natural", R=777, K=300,
             S=5, beta1=4.0, beta_adapt=1, population=True),
        # The headline solve: G63's size, full schedule, every part of the
        # method on.
        dict(name="g63-7000", kind="random", n=7000, m=41459, signed=False, order="natural", R=4096, K=2000,
             S=10, beta1=5.0, as_enable=1, nl_period=10),
        # The same graph with single-replica cluster updates, a tenth of the
        # schedule, colouring order (few, large dependency levels).
        dict(name="wolff-7000", kind="random", n=7000, m=41459, signed=False, order="coloring", R=4096, K=200,
             S=10, beta1=5.0, as_enable=1, nl_period=10, nl_kind=1),
        # Toroidal family, the benchmark's second workload with a fifth of its steps.
        dict(name="torus-100", kind="torus", L=100, signed=True, order="checkerboard", R=16384, K=200, S=5,
             beta1=4.0),
        # The largest graphs: a 140 x 140 torus.
        dict(name="torus-140", kind="torus", L=140, signed=True, order="checkerboard", R=8192, K=100, S=5,
             beta1=4.0),
        # A batch of uneven instances sharing launches.
        dict(name="batch-16", kind="batch", count=16, mix=5, K=100),
        # A queue of requests served by the resident pool, graphs validated
        # and runs planned inside the pass.
        dict(name="serve-16", kind="serve", count=16, mix=6, K=100),
    ]


def _log_int(rng, lo, hi) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# Attempts (R N S K) of a drawn single run at most; the headline solve has 5.7e11.
_MOST_ATTEMPTS = 3e10


def draw(rng) -> dict:
    u = rng.random()
    if u < 0.12:
        return dict(kind="batch", count=_log_int(rng, 2, 24), mix=rng.randrange(1 << 20), K=_log_int(rng, 20, 120))
    if u < 0.24:
        return dict(kind="serve", count=_log_int(rng, 2, 24), mix=rng.randrange(1 << 20), K=_log_int(rng, 20, 120))
    signed = rng.random() < 0.5
    c = dict(signed=signed, R=_log_int(rng, 64, 16384), K=_log_int(rng, 10, 300), S=rng.choice([1, 3, 5, 10, 20]),
             beta1=round(rng.uniform(1.0, 5.0), 2))
    if u < 0.45:
        c.update(kind="torus", L=_log_int(rng, 5, 141), order="checkerboard")
        if c["L"] & 1:
            c["order"] = rng.choice(["natural", "random"])
        n = c["L"] * c["L"]
    else:
        n = _log_int(rng, 20, 20000)
        # Mean degrees from 2 on sparse graphs to 48, and to 200 on small ones.
        most = min(200.0 if n <= 1500 else 48.0 if n <= 3000 else 14.0, (n - 1) / 2.0)
        d = math.exp(rng.uniform(math.log(2.0), math.log(most)))
        c.update(kind="random", n=n, m=max(1, int(n * d / 2)), order=rng.choice(["natural", "natural", "coloring", "random"]))
    if c["kind"] == "random" and c["n"] > 12000:
        c["signed"] = False
    if rng.random() < 0.5:
        c["as_enable"] = 1
    v = rng.random()
    if v < 0.25:
        c.update(nl_period=rng.choice([1, 5, 10]), nl_kind=0)
        c["R"] += c["R"] & 1
    elif v < 0.4:
        c.update(nl_period=rng.choice([5, 10]), nl_kind=1)
    if rng.random() < 0.2:
        c["beta_adapt"] = 1
    cost = float(c["R"]) * n * c["S"]
    c["K"] = max(4, min(c["K"], int(_MOST_ATTEMPTS / cost)))
    if float(c["R"]) * n <= 4e6 and rng.random() < 0.5:
        c["population"] = True
    return c


def _graph(c, seed):
    if c["kind"] == "torus":
        return W.torus(c["L"], seed, c["signed"])
    g = W.random_graph(c["n"], c["m"], seed)
    if c["signed"]:
        i, j, _ = g.edges()
        sign = 1 - 2 * (W.splitmix64(seed + 1, len(i)) & np.uint64(1)).astype(np.int64)
        g = W.from_edges(g.n, i, j, sign)
    return g


def _order(c, g, seed):
    if c["order"] == "checkerboard":
        return W.checkerboard_order(c["L"])
    if c["order"] == "coloring":
        return W.coloring_order(g)
    if c["order"] == "random":
        return np.random.default_rng(seed).permutation(g.n).astype(np.int32)
    return W.natural_order(g.n)


def _mix(c, seed):
    """The instances of a batch or a queue: sizes and schedules of the case's
    mix, graphs and run seeds from ``seed``."""
    make = W.batch_workloads if c["kind"] == "batch" else W.serve_requests
    out = []
    for j, w in enumerate(make(c["count"], meta_seed=c["mix"], steps=c["K"])):
        g = w["graph"]
        if "torus" in g.name:
            g = W.torus(math.isqrt(g.n), seed + j, True)
        else:
            g = W.random_graph(g.n, g.n_edges, seed + j)
        out.append(dict(w, graph=g, seed=seed))
    return out


def prepare(case, seed):
    """What a program holds before the call: validated graphs and run
    parameters, for the batch its plan, for the server its request queue."""
    c = case
    if c["kind"] == "batch":
        wls = _mix(c, seed)
        solvers = [pa.Solver(w["graph"]) for w in wls]
        return dict(case=c, solvers=solvers,
                    batch=pa.FusedBatch(solvers, [pa.params_from_workload(w) for w in wls]))
    if c["kind"] == "serve":
        return dict(case=c, server=serve.PoolServer(hbm_budget=4 << 30),
                    requests=[serve.Request(i, w["graph"], pa.params_from_workload(w))
                              for i, w in enumerate(_mix(c, seed))])
    g = _graph(c, seed)
    p = pa.RunParams(betas=W.linear_betas(0.1, c["beta1"], c["K"]), sweeps=c["S"], R=c["R"], seed=seed,
                     inst=seed % 65536, order=_order(c, g, seed), as_enable=c.get("as_enable", 0),
                     nl_period=c.get("nl_period", 0), nl_kind=c.get("nl_kind", 0),
                     beta_adapt=c.get("beta_adapt", 0))
    return dict(case=c, solver=pa.Solver(g), params=p)


def _results(s, population):
    out = dict(cut=s.best_cut(), best=s.best_info(), x=s.best_config(), stats=s.step_stats())
    if population:
        out["pop_x"], out["pop_E"] = s.population()
    return out


def run(state):
    """One pass: the whole call and the results a caller reads."""
    c = state["case"]
    if c["kind"] == "batch":
        state["batch"].run()
        res = [_results(s, False) for s in state["solvers"]]
        return dict(cut=np.array([r["cut"] for r in res]),
                    best=np.array([list(r["best"].values()) for r in res]),
                    x=np.concatenate([r["x"] for r in res]), stats=np.stack([r["stats"] for r in res]))
    if c["kind"] == "serve":
        res = sorted(state["server"].serve(state["requests"], realtime=False), key=lambda r: r.rid)
        return dict(cut=np.array([r.best_cut for r in res]),
                    best=np.array([list(r.best_info.values()) for r in res]),
                    x=np.concatenate([r.best_x for r in res]), stats=np.stack([r.stats for r in res]))
    state["solver"].run(state["params"])
    return _results(state["solver"], c.get("population", False))


def exact(case, seed):
    return None


def _mean_run(c):
    """(nodes, edges, replicas, sweeps, steps) of a run of the case; for a
    batch or a queue the mean over its instance mix, times their count."""
    if c["kind"] == "torus":
        return c["L"] ** 2, 2 * c["L"] ** 2, c["R"], c["S"], c["K"], 1
    if c["kind"] == "random":
        return c["n"], c["m"], c["R"], c["S"], c["K"], 1
    if c["kind"] == "batch":        # N ~ U[800, 7000], R ~ U[256, 4096], 10 or 5 sweeps
        return 3900, 11700, 2176, 7.5, c["K"], c["count"]
    return 5965, 16000, 2770, 5, c["K"], c["count"]     # log-uniform N in [800, 20000], R in [512, 8192]


def work(case):
    """Bytes: the graph read once, the best configuration and the statistics
    (and the population where it is asked for) written once; the method's
    state fits the chip, so no more has to move. Operations: the method's own
    32-bit integer operations, per attempt one add per neighbour, six for the
    test, flip and energy, and a quarter of a Philox4x32-10 call (25) where a
    move is uphill, as nine in ten are. Adaptive runs take about a third of
    their grid points."""
    n, m, R, S, K, count = _mean_run(case)
    steps = K / 3.0 if case.get("beta_adapt") else K
    out = n + 80.0 * K + (float(R) * (n + 4) if case.get("population") else 0.0)
    return {"bytes": count * (4.0 * (n + 1) + 10.0 * m + out),
            "flops": count * float(R) * n * S * steps * (2.0 * m / n + 6 + 25 * 0.9)}
