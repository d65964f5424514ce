"""The tile sweep form at the edges of its rows, counters, records and draw
buffer, bit-exact against the CPU oracle."""
import numpy as np
import pytest

from paper_2510_21105_amd import workloads as W
from tests.test_gpu_parity import _check_against_oracle, _compare, _cycle_with_hub, pa  # noqa: F401

pytestmark = pytest.mark.gpu


def _hub(n, deg, signed):
    g = _cycle_with_hub(n, deg)
    if not signed:
        i, j, _ = g.edges()
        g = W.from_edges(g.n, i, j, np.ones(len(i), np.int64), g.name + "u")
    return g


# Rows end after 4 or 6, 14 and 22 entries, lanes per node double past them,
# the counters widen after degrees 63 and 127; 1,024 is past the form's range.
@pytest.mark.parametrize("deg", [4, 5, 6, 7, 8, 9, 14, 15, 16, 17, 22, 23, 63, 64, 127, 128, 352, 353, 1023, 1024])
@pytest.mark.parametrize("signed", [False, True])
def test_row_and_counter_edges(pa, deg, signed):  # noqa: F811
    g = _hub(max(40, deg + 37), deg, signed)
    wl = dict(W.workload("small800"), graph=g, R=37, betas=W.linear_betas(0.02, 1.5, 4), sweeps=2,
              order=W.natural_order(g.n), nl_period=0)
    s, _ = _compare(pa, g, wl, record=0)
    assert s.launch_info()["sweep_kernel"] == (1 if deg <= 1023 else 2)


# Nodes: one item, a full one, one lane more; more than half the draw buffer
# (chunks change inside a sweep). Replicas: a part of a tile, several words.
# Betas: tables whose buckets hold one threshold, many, or accept everything.
@pytest.mark.parametrize("tile", [0, 4, 8, 16])
@pytest.mark.parametrize("n,m,R,threads,signed", [
    (2, 1, 1, 0, False), (64, 160, 3, 64, False), (65, 400, 130, 64, True), (129, 1900, 70, 1024, False),
    (3000, 9000, 20, 128, True), (4000, 30000, 16, 0, False)])
def test_items_chunks_and_tiles(pa, tile, n, m, R, threads, signed):  # noqa: F811
    g = W.random_graph(n, m, 5 + n, f"r{n}")
    if signed:
        i, j, _ = g.edges()
        g = W.from_edges(n, i, j, 1 - 2 * (np.arange(len(i)) % 3 == 0).astype(np.int64), f"s{n}")
    wl = dict(W.workload("small800"), graph=g, R=R, betas=[0.0, 1e-5, 0.01, 0.4, 2.0], sweeps=3,
              order=W.natural_order(n), nl_period=0)
    _compare(pa, g, wl, dict(tile_replicas=tile, wg_threads=threads), record=1)


# Draws in registers (regular, few levels): full and ragged last items of a
# level, an odd count of them, more items than the sums hold between flushes.
@pytest.mark.parametrize("L,R,signed,tile", [(32, 9, True, 0), (46, 17, False, 0), (62, 40, True, 4),
                                             (98, 12, False, 8), (34, 33, True, 8)])
def test_large_levels_draw_in_registers(pa, L, R, signed, tile):  # noqa: F811
    g = W.torus(L, 7, signed)
    wl = dict(W.workload("torus100"), graph=g, R=R, betas=[0.0, 0.05, 0.7, 3.0], sweeps=3,
              order=W.checkerboard_order(L))
    _compare(pa, g, wl, dict(tile_replicas=tile, wg_threads=64 if L == 98 else 0), record=1)


# Degree 2: one threshold, two padding neighbours. Even nodes, then odd ones.
@pytest.mark.parametrize("n,R,signed", [(514, 5, False), (1300, 40, True)])
def test_rings_draw_in_registers(pa, n, R, signed):  # noqa: F811
    i = np.arange(n)
    w = 1 - 2 * ((i % 5 == 0) & signed).astype(np.int64)
    g = W.from_edges(n, i, (i + 1) % n, w, f"ring{n}")
    order = np.concatenate([i[::2], i[1::2]]).astype(np.int32)
    wl = dict(W.workload("torus100"), graph=g, R=R, betas=[0.0, 0.3, 2.0], sweeps=3, order=order)
    _compare(pa, g, wl, record=1)


def test_workspace_without_room_for_the_tile_plan(pa):  # noqa: F811
    """A workspace that only the general form's plan fits is still enough."""
    import torch
    L = 20
    g = W.torus(L, 3, True)
    wl = dict(W.workload("torus100"), graph=g, R=40, betas=[0.2, 0.9, 2.0], sweeps=2, order=W.natural_order(g.n))
    p = pa.params_from_workload(wl)
    s, t = pa.Solver(g), pa.Solver(g)
    need = s.workspace_bytes(p)
    s.run(p)
    t.run(p, workspace=torch.empty(need - 256, dtype=torch.uint8, device="cuda"))
    assert s.launch_info()["lds_bytes"] != t.launch_info()["lds_bytes"]
    for a, b in zip(s.population(), t.population()):
        assert np.array_equal(a, b)
    assert np.array_equal(s.step_stats(), t.step_stats()) and s.best_info() == t.best_info()


def test_shared_launches(pa):  # noqa: F811
    """Fused runs of one record mode and size class: degrees up to 100 (wide
    counters for the whole group), small levels, a regular and a ragged
    signed graph, before and after the shape is tuned."""
    gs = [(_hub(300, 100, False), 33), (W.random_graph(700, 2800, 3, "f1"), 70), (_hub(500, 40, True), 9),
          (W.torus(30, 5, True), 130), (W.torus(24, 6, True), 17)]
    wls = [dict(W.workload("small800"), graph=g, R=R, betas=[0.0, 0.1, 0.8, 2.0][:k], sweeps=2, nl_period=0,
                inst=q, order=W.checkerboard_order(int(g.n ** 0.5)) if "torus" in g.name else W.natural_order(g.n))
           for q, ((g, R), k) in enumerate(zip(gs, (4, 3, 4, 2, 4)))]
    params = [pa.params_from_workload(w, record=3) for w in wls]
    solvers = [pa.Solver(w["graph"]) for w in wls]
    fb = pa.FusedBatch(solvers, params)
    fb.run()
    for w, p, s in zip(wls, params, solvers):
        _check_against_oracle(s, w, p)
    fb.tune(probe_steps=1)
    fb.run()
    for w, p, s in zip(wls, params, solvers):
        _check_against_oracle(s, w, p)


def test_pool_without_room_for_the_tile_plan(pa):  # noqa: F811
    """The smallest pool that takes a run steps it in the general form."""
    import torch
    L = 20
    g = W.torus(L, 3, True)
    wl = dict(W.workload("torus100"), graph=g, R=40, betas=[0.2, 0.9, 2.0], sweeps=2, order=W.natural_order(g.n))
    p = pa.params_from_workload(wl)
    s, t = pa.Solver(g), pa.Solver(g)
    s.run(p)
    mem = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")

    def takes(size):
        try:
            pool = pa.Pool(workspace=(mem.data_ptr(), size))
            pool.submit(t, p)
        except pa.PAError:
            return None
        return pool

    lo, hi = 1, (64 << 20) // 256
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if takes(256 * mid) else (mid, hi)
    for size, general in ((256 * hi, True), (64 << 20, False)):
        pool = takes(size)
        while not pool.advance(iterations=8):
            pass
        torch.cuda.synchronize()
        assert len(pool.poll()) == 1
        assert (t.launch_info()["lds_bytes"] < 16384) == general
        for a, b in zip(s.population(), t.population()):
            assert np.array_equal(a, b)
        assert np.array_equal(s.step_stats(), t.step_stats()) and s.best_info() == t.best_info()
        pool.close()
