"""Which launch shape and sweep form a run takes, alone, in a fused batch or in
the pool, and the forms that only some runs take, against the CPU oracle.

The two forms of kernel 1 are told apart by the LDS of a workgroup: the tile
form's records start at byte 20,360 (256 where it draws in registers)."""
import numpy as np
import pytest

from paper_2510_21105_amd import workloads as W
from tests.test_gpu_parity import _check_against_oracle, _compare, pa  # noqa: F401

pytestmark = pytest.mark.gpu


def _two_levels(n, deg, signed):
    """Natural order gives two levels of n / 2 nodes: a ring between the halves
    and node 0 joined to deg nodes of the second half. Not regular."""
    h = n // 2
    i = np.arange(h)
    pairs = {(int(a), int(b)) for a, b in zip(np.r_[i, i], np.r_[h + i, h + (i + 1) % h])}
    far = np.linspace(2, h - 2, deg - 2).round().astype(int) if deg > 2 else []
    pairs |= {(0, h + int(t)) for t in far}
    e = np.array(sorted(pairs))
    w = 1 - 2 * ((np.arange(len(e)) % 3 == 0) & signed).astype(np.int64)
    g = W.from_edges(n, e[:, 0], e[:, 1], w, f"two{n}d{deg}{'s' if signed else ''}")
    assert int(g.degrees().max()) == deg
    return g


def _wl(g, R, betas, sweeps=2, **over):
    return dict(W.workload("small800"), graph=g, R=R, betas=list(betas), sweeps=sweeps,
                order=W.natural_order(g.n), nl_period=0, desc=f"{g.name} R={R}", **over)


def _byte_lds(n, tile, copies=False):
    return 1024 + (((2 * n if copies else n) + 1) * tile + 15 & ~15) + 384


@pytest.mark.parametrize("tune", [False, True])
@pytest.mark.parametrize("R,byte", [(2040, False), (2057, True), (4096, True), (4104, False)])
def test_fused_batch_keeps_the_byte_form_on_large_levels(pa, R, byte, tune):  # noqa: F811
    """Up to two 8-replica workgroups a compute unit on levels of more than 480
    nodes: the form that a run alone takes there, untuned; a tuned batch may
    take either. Results are the oracle's with both."""
    g = _two_levels(1000, 13, True)
    wl = _wl(g, R, (0.1, 0.8, 1.9))
    p = pa.params_from_workload(wl, record=3)
    s = pa.Solver(g)
    fb = pa.FusedBatch([s], [p])
    if tune:
        fb.tune(probe_steps=1)
    else:
        assert (fb.info()[0]["lds_bytes"] == _byte_lds(1000, 8)) == byte, fb.info()
    fb.run()
    _check_against_oracle(s, wl, p)

def _pooled(pa, wls):
    """The runs submitted together to one pool and stepped to the end: their solvers."""
    import torch
    pool = pa.Pool(256 << 20)
    stream = torch.cuda.Stream()
    solvers = [pa.Solver(w["graph"]) for w in wls]
    for s, w in zip(solvers, wls):
        pool.submit(s, pa.params_from_workload(w, record=3))
    while pool.info()["waiting"] or pool.info()["stepping"]:
        pool.advance(stream, 4)
    torch.cuda.synchronize()
    assert len(pool.poll()) == len(wls)
    out = []
    for s, w in zip(solvers, wls):
        _check_against_oracle(s, w, pa.params_from_workload(w, record=3))
        out.append(s.launch_info())
    pool.close()
    return out

def test_pooled_run_takes_threads_by_the_load(pa):  # noqa: F811
    """A run alone in the pool whose workgroups get a compute unit each takes
    more threads than the same run among many; in between, on large levels, the
    byte form. Results are the oracle's every time."""
    g = _two_levels(1000, 13, False)
    few = [_wl(g, 100, (0.1, 0.9, 2.0), inst=q) for q in range(2)]
    alone = _pooled(pa, few[:1])[0]
    both = _pooled(pa, [few[0], _wl(W.torus(12, 3, True), 2500, (0.1,), sweeps=1)])[0]
    crowd = _pooled(pa, [few[1], _wl(W.torus(12, 3, True), 6000, (0.1,), sweeps=1)])[0]
    assert both["lds_bytes"] == _byte_lds(1000, 8) < min(alone["lds_bytes"], crowd["lds_bytes"])
    assert alone["threads"] > crowd["threads"]


@pytest.mark.parametrize("R,jump", [(512, 64), (513, 17), (513, 18), (2048, 10), (2049, 9), (2049, 10), (8193, 64)])
def test_adaptive_jumps_at_every_epilogue_width(pa, R, jump):  # noqa: F811
    """One wave tries one jump: 8 or 16 waves, in one pass and in several."""
    g = W.random_graph(40, 120, 3)
    wl = _wl(g, R, np.linspace(0.05, 3.2, 80), beta_adapt=1, adapt_jump=jump)
    _compare(pa, g, wl, record=0)
