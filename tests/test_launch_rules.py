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
    """Two 8-replica workgroups a compute unit on levels of work enough for all
    waves: the form that a run alone takes there, untuned; a tuned batch may
    take either. Results are the oracle's with both."""
    g = _two_levels(2000, 13, True)
    wl = _wl(g, R, (0.1, 0.8, 1.9))
    p = pa.params_from_workload(wl, record=3)
    s = pa.Solver(g)
    fb = pa.FusedBatch([s], [p])
    if tune:
        fb.tune(probe_steps=1)
    else:
        assert (fb.info()[0]["lds_bytes"] == _byte_lds(2000, 8)) == byte, fb.info()
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
    more threads than the same run among many; with two a unit and large levels
    it takes the byte form. Results are the oracle's every time."""
    g = _two_levels(2000, 13, False)
    few = [_wl(g, 100, (0.1, 0.9, 2.0), inst=q) for q in range(2)]
    t, betas = W.torus(12, 3, True), np.linspace(0.1, 1.0, 10)
    alone = _pooled(pa, few[:1])[0]
    both = _pooled(pa, [few[0], _wl(t, 2500, betas, sweeps=6)])[0]
    crowd = _pooled(pa, [few[1], _wl(t, 6000, betas, sweeps=6)])[0]
    assert both["lds_bytes"] == _byte_lds(2000, 8) < min(alone["lds_bytes"], crowd["lds_bytes"])
    assert alone["threads"] > crowd["threads"]
    # Runs that end long before it leave it alone for most of its time.
    short = _pooled(pa, [few[0], _wl(t, 2500, (0.1,), sweeps=1)])[0]
    assert (short["threads"], short["lds_bytes"]) == (alone["threads"], alone["lds_bytes"])


@pytest.mark.parametrize("signed", [False, True])
def test_pooled_tori_draw_in_registers(pa, signed):  # noqa: F811
    """Regular graphs of few levels step in the pool without a draw buffer."""
    wls = [dict(_wl(W.torus(L, 5 + L, signed), R, (0.0, 0.4, 1.5), sweeps=3, inst=L),
                order=W.checkerboard_order(L)) for L, R in ((32, 70), (46, 9))]
    for w, info in zip(wls, _pooled(pa, wls)):
        assert info["lds_bytes"] < 256 + 4 * (w["graph"].n + 32), info


@pytest.mark.parametrize("R,jump", [(512, 64), (513, 17), (513, 18), (2048, 10), (2049, 9), (2049, 10), (8193, 64)])
def test_adaptive_jumps_at_every_epilogue_width(pa, R, jump):  # noqa: F811
    """One wave tries one jump: 8 or 16 waves, in one pass and in several."""
    g = W.random_graph(40, 120, 3)
    wl = _wl(g, R, np.linspace(0.05, 3.2, 80), beta_adapt=1, adapt_jump=jump)
    _compare(pa, g, wl, record=0)


# Automatic runs that keep the byte form (two 8-replica workgroups a compute
# unit on large levels): rows of every register count, unsigned records and
# complemented copies, offsets and (above 8,063 nodes) indices as entries.
@pytest.mark.parametrize("n,deg,R,signed", [
    (2000, 5, 2049, False), (2000, 8, 3001, True), (2000, 13, 4090, False), (2000, 14, 4096, True),
    (2000, 21, 4090, True), (2000, 22, 4096, False), (2000, 30, 4096, True), (2000, 33, 4090, False),
    (8200, 8, 2100, False)])
def test_byte_form_on_large_levels(pa, n, deg, R, signed):  # noqa: F811
    g = _two_levels(n, deg, signed)
    s, _ = _compare(pa, g, _wl(g, R, (0.0, 0.3, 1.7), sweeps=2 if n == 2000 else 1), record=0)
    info = s.launch_info()
    assert info["sweep_kernel"] == 1 and info["tile_replicas"] == 8
    assert info["lds_bytes"] == _byte_lds(n, 8, signed), info


# One block row a level to either side of the line, and a degree to either
# side: the other form.
@pytest.mark.parametrize("n,deg,byte", [(1792, 6, False), (1794, 6, True), (2000, 33, True), (2000, 34, False),
                                        (4000, 42, True), (4000, 43, False)])
def test_form_by_rows_a_level_and_degree(pa, n, deg, byte):  # noqa: F811
    g = _two_levels(n, deg, False)
    s = pa.Solver(g)
    s.run(pa.params_from_workload(_wl(g, 4096, (0.2,), sweeps=1)))
    assert (s.launch_info()["lds_bytes"] == _byte_lds(n, 8)) == byte, s.launch_info()


def test_byte_form_on_the_benchmark_graph_in_colouring_order(pa):  # noqa: F811
    """7,000 nodes, R = 4,096, ten levels: the byte form with issue turns."""
    base = W.workload("g63like")
    g = base["graph"]
    wl = dict(base, order=W.coloring_order(g), betas=base["betas"][100:103], sweeps=2, nl_period=2, nl_kind=1)
    s, _ = _compare(pa, g, wl, record=0)
    info = s.launch_info()
    assert info["levels"] <= 14 and info["lds_bytes"] == _byte_lds(7000, 8), info


def _ring_rows(n, deg, signed):
    """Every node joined to its deg / 2 nearest on either side (deg even)."""
    i = np.arange(n)
    a = np.concatenate([i] * (deg // 2))
    b = np.concatenate([(i + k) % n for k in range(1, deg // 2 + 1)])
    w = 1 - 2 * ((np.arange(len(a)) % 3 == 0) & signed).astype(np.int64)
    return W.from_edges(n, a, b, w, f"rows{deg}{'s' if signed else ''}")


# The byte form where a workspace has no room for the tile form's plan (even
# rows of many lanes make that the larger one): every tile width, rows in
# registers, rows past them, the largest degree.
@pytest.mark.parametrize("tile", [4, 8, 16])
@pytest.mark.parametrize("deg,signed", [(12, False), (18, True), (30, False), (32, False), (32, True), (64, False),
                                        (126, False)])
def test_byte_form_in_a_small_workspace(pa, tile, deg, signed):  # noqa: F811
    import torch
    g = _ring_rows(400, deg, signed)
    wl = _wl(g, 37, (0.05, 0.9))
    p = pa.params_from_workload(wl, record=3, tile_replicas=tile)
    s = pa.Solver(g)
    need = s.workspace_bytes(p)
    s.run(p, workspace=torch.empty(need - 256, dtype=torch.uint8, device="cuda"))
    info = s.launch_info()
    assert info["tile_replicas"] == tile and info["lds_bytes"] == _byte_lds(400, tile, signed), info
    _check_against_oracle(s, wl, p)


@pytest.mark.parametrize("n,R,signed", [(514, 5, False), (1300, 40, True)])
def test_rings_of_eight_replicas_draw_in_registers(pa, n, R, signed):  # noqa: F811
    """Degree 2 in the nibble test: one threshold, two padding neighbours."""
    i = np.arange(n)
    g = W.from_edges(n, i, (i + 1) % n, 1 - 2 * ((i % 5 == 0) & signed).astype(np.int64), f"ring{n}")
    wl = dict(_wl(g, R, (0.0, 0.3, 2.0), sweeps=3), order=np.concatenate([i[::2], i[1::2]]).astype(np.int32))
    s, _ = _compare(pa, g, wl, dict(tile_replicas=8), record=1)
    assert s.launch_info()["tile_replicas"] == 8 and s.launch_info()["lds_bytes"] < 256 + 4 * (n + 32)
