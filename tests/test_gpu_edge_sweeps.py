"""Edge sweeps -- both products of a power step in one pass, edge by edge -- against the oracle: every split of
rows over threads, one and many row blocks, short rows, vectors of every length class, dropped columns."""
import numpy as np
import pytest

from oracle import pg_oracle as O
from parity_util import TOL_1, TOL_10, compare_state, env_setting, env_settings, graph_workload, launched, oracle_problem, oracle_rounds

pytestmark = pytest.mark.gpu

# one thread to a whole work-group per row, one to five units per thread, every remainder of q modulo 4, fewer rows than a step
# takes and several row blocks, rows of one to three floats, vectors for one wavefront and for many
SHAPES = [(300, 576), (33, 130), (517, 259), (50, 4609), (40, 3000), (1030, 36), (9, 3), (4100, 2), (700, 1), (5000, 1), (1, 77),
          (1, 1), (7, 8), (130, 1024), (20, 2306), (4, 4), (64, 17), (3, 640), (21, 12001)]
WIDE = [(140, 7001), (30, 650), (90, 1), (9, 5121), (600, 5), (11, 25002)]     # rows that take work-groups of 512
GRAPHS = {"ring": (5, [(0, 1), (1, 2), (2, 3), (3, 4), (4, 0)]),
          "path and a lone worker": (4, [(1, 0), (1, 2)]),
          "hub": (6, [(0, 1), (2, 0), (0, 3), (4, 0), (3, 5)])}


def _workload(graph, shapes, rank, steps, seed=41):
    return graph_workload(f"sweep {graph} {len(shapes)} r{rank}", GRAPHS[graph], shapes, rank, steps, seed)


def _buffers(wl, X, Q):
    from paper_2008_01425_amd.device import GossipBuffers
    with env_setting("PG_EDGE", 0), env_setting("PG_SWEEP", 1):
        gb = GossipBuffers.from_workload(wl, fill=False)
    gb.fill_from_arrays(X, Q)
    return gb


@pytest.mark.parametrize("graph", GRAPHS)
@pytest.mark.parametrize("rank,steps", [(1, 1), (2, 2), (3, 1), (4, 1)])
@pytest.mark.parametrize("wide", [False, True])
def test_rounds_runs_and_gradients_against_the_oracle(graph, rank, steps, wide):
    shapes = WIDE if wide else SHAPES
    wl = _workload(graph, shapes, rank, steps)
    layers = list(range(len(wl.shapes)))
    prob = oracle_problem(wl)
    X, Q = wl.all_params(), wl.all_q()
    for l in (0, 1, 2):                               # two neighbours agree: their columns are dropped
        X[1][l] = X[0][l].copy()
    print(f"case {wl.name}", flush=True)
    a, b, c, d = (_buffers(wl, X, Q) for _ in range(4))
    kinds = launched(a, a.round)
    assert kinds["edge_sweep"] == steps and kinds["finish"] == steps and "sweep_p" not in kinds, kinds
    kinds = launched(b, lambda: b.run(3))
    assert kinds["edge_sweep"] == 3 * steps, kinds
    c.run(4)
    rng = np.random.default_rng(5)
    G = [[rng.standard_normal(s).astype(np.float32) for s in wl.shapes] for _ in range(wl.n_workers)]
    d.alloc_grads()
    for i in range(wl.n_workers):
        for l in layers:
            d.set_grad_layer(i, l, G[i][l])
    d.round_sgd(0.05)
    Xg, Qg = [[x.copy() for x in w] for w in X], [[q.copy() for q in e] for e in Q]
    O.gossip_round(prob, Xg, Qg, G=G, eta=float(np.float32(0.05)))
    compare_state(d, Xg, Qg, layers, TOL_1, what="sgd " + wl.name)
    info, snaps = oracle_rounds(wl, X, Q, 4, layers, snap_at=(1, 3))
    compare_state(a, snaps[1].X, snaps[1].Q, layers, TOL_1, what="round", phat=snaps[1].phat, flags=snaps[1].degenerate)
    # (Phat is compared after one round: the column sums of a large layer are formed before it is rounded, and after a few
    # rounds on 30 rows what is left of the difference reacts to that by more than the ten-round bar)
    compare_state(b, snaps[3].X, snaps[3].Q, layers, TOL_10, what="run of 3", flags=snaps[3].degenerate)
    compare_state(c, X, Q, layers, TOL_10, what="run of 4", flags=info.degenerate)
    for _ in range(3):                                # a run is its rounds, bit for bit
        a.round()
    assert all(bool((x == y).all()) for x, y in zip(a.x, c.x)) and bool((a.q == c.q).all())
    for gb in (a, b, c, d):
        gb.close()


@pytest.mark.parametrize("graph", GRAPHS)
@pytest.mark.parametrize("rank", [1, 2, 4])
@pytest.mark.parametrize("wide", [False, True])
def test_update_in_one_launch_is_the_row_kernels_update(graph, rank, wide):
    """Same operations in the same order: bit for bit, with and without gradients, on every length of row and remainder of four."""
    wl = _workload(graph, WIDE if wide else SHAPES, rank, 1, seed=43)
    X, Q = wl.all_params(), wl.all_q()
    rng = np.random.default_rng(6)
    G = [[rng.standard_normal(s).astype(np.float32) for s in wl.shapes] for _ in range(wl.n_workers)]
    print(f"case {wl.name}", flush=True)
    got, launches = [], []
    for mixed in (0, 1):
        with env_setting("PG_MIXED", mixed):
            gb = _buffers(wl, X, Q)
        gb.alloc_grads()
        for i in range(wl.n_workers):
            for l in range(len(wl.shapes)):
                gb.set_grad_layer(i, l, G[i][l])
        kinds = launched(gb, gb.round)
        launches.append(kinds["update"])
        gb.round_sgd(0.05)
        gb.run(2)
        got.append(gb)
    assert launches[1] == 1 <= launches[0], launches
    a, b = got
    assert all(bool((x == y).all()) for x, y in zip(a.x, b.x)) and bool((a.q == b.q).all())
    a.close()
    b.close()


def test_overflow_stays_where_it_is():
    """Columns that overflow a float (differences of 3e37, sums over 400 rows; P itself fits) reach the entries that the row kernels' update gives them, on workers with fewer columns too."""
    from paper_2008_01425_amd.device import GossipBuffers
    wl = _workload("hub", [(400, 5), (900, 4)], 1, 1, seed=47)
    X, Q = wl.all_params(), wl.all_q()
    X = [[np.full_like(x, -1.5e37 if i in (1, 2, 3, 4) else 1.5e37) for x in w] for i, w in enumerate(X)]
    got = []
    for edge, sweep, mixed in ((0, 0, 0), (0, 1, 0), (0, 1, 1), (1, 0, 0)):
        print(f"edge {edge} sweep {sweep} mixed {mixed}", flush=True)
        with env_setting("PG_EDGE", edge), env_setting("PG_SWEEP", sweep), env_setting("PG_MIXED", mixed):
            gb = GossipBuffers.from_workload(wl, fill=False)
        gb.fill_from_arrays(X, Q)
        gb.round()
        got.append([x.cpu().numpy().copy() for x in gb.x])
        gb.close()
    assert any(np.isinf(x).any() for x in got[0])
    for other in got[1:]:
        for x, y in zip(got[0], other):
            assert (np.isnan(x) == np.isnan(y)).all() and (np.isinf(x) == np.isinf(y)).all()


@pytest.mark.parametrize("rank", [1, 2, 3])
@pytest.mark.parametrize("place", ["last", "inside the last unit", "first"])
def test_an_infinite_parameter_spreads_as_it_does_with_the_row_kernels(rank, place):
    """A unit that is moved back to the row's end, and threads past it, load floats that are others' own: an infinity there must not
    turn the products into NaN and drop the columns.  Rows of every remainder of four, with and without idle units, walked once and twice."""
    from paper_2008_01425_amd.device import GossipBuffers
    shapes = [(100, 130), (300, 577), (64, 4610), (70, 1151), (2100, 5), (33, 131), (40, 17), (9, 7), (21, 12001), (5000, 3), (90, 128), (60, 4608),
              (700, 1), (20, 642)]
    wl = _workload("hub", shapes, rank, 1, seed=53)
    X, Q = wl.all_params(), wl.all_q()
    for l, (p, q) in enumerate(shapes):
        X[1][l][p // 2, {"last": q - 1, "inside the last unit": max(0, q - 3), "first": 0}[place]] = np.inf if l % 2 else -np.inf
    got = []
    for sweep in (0, 1):
        print(f"rank {rank} {place} sweep {sweep}", flush=True)
        with env_setting("PG_EDGE", 0), env_setting("PG_SWEEP", sweep):
            gb = GossipBuffers.from_workload(wl, fill=False)
        gb.fill_from_arrays(X, Q)
        gb.round()
        got.append(gb)
    a, b = got
    for l in range(len(shapes)):
        for e in range(wl.n_edges):
            assert np.array_equal(a.get_flags(e, l), b.get_flags(e, l)), (shapes[l], "flags", e)
            assert np.array_equal(np.isfinite(a.get_q(e, l)), np.isfinite(b.get_q(e, l))), (shapes[l], "state", e)
        for i in range(wl.n_workers):
            x, y = a.get_layer(i, l), b.get_layer(i, l)
            assert np.array_equal(np.isnan(x), np.isnan(y)) and np.array_equal(np.isinf(x), np.isinf(y)), (shapes[l], "worker", i)
    a.close()
    b.close()


@pytest.mark.parametrize("graph", ["ring", "path and a lone worker"])
@pytest.mark.parametrize("rank", [1, 2])
def test_runs_that_write_every_second_round_are_their_rounds(graph, rank):
    """Sets that qualify for both: a run of any length, its rounds one by one and runs of one round leave the same, bit for
    bit; the SGD round, which no run contains, takes the sweeps."""
    from paper_2008_01425_amd.device import GossipBuffers
    wl = _workload(graph, [(64, 576), (33, 130), (517, 259), (50, 4609), (1030, 36), (700, 1), (1, 77), (7, 8)], rank, 1, seed=59)
    X, Q = wl.all_params(), wl.all_q()
    got, kinds = [], []
    calls = {"run": lambda gb: gb.run(3), "rounds": lambda gb: [gb.round() for _ in range(3)], "runs of two and one": lambda gb: (gb.run(2), gb.run(1))}
    for what, call in calls.items():
        print(f"case {wl.name} {what}", flush=True)
        with env_setting("PG_EDGE", 0), env_setting("PG_LIGHT", 0), env_setting("PG_LAZY", 1), env_setting("PG_SWEEP", 1):
            gb = GossipBuffers.from_workload(wl, fill=False)
        gb.fill_from_arrays(X, Q)
        kinds.append(launched(gb, lambda: call(gb)))
        got.append(gb)
    assert "peek_sweep_p" in kinds[0] and "peek_sweep_p" in kinds[2] and all("edge_sweep" not in k for k in kinds), kinds
    for other in got[1:]:
        assert all(bool((x == y).all()) for x, y in zip(got[0].x, other.x)) and bool((got[0].q == other.q).all())
    info = oracle_rounds(wl, X, Q, 3, list(range(len(wl.shapes))))
    compare_state(got[0], X, Q, list(range(len(wl.shapes))), TOL_10, what="run of 3", flags=info.degenerate)
    got[0].alloc_grads()
    for g in got[0].g:
        g.zero_()
    assert "edge_sweep" in launched(got[0], lambda: got[0].round_sgd(0.0))
    for gb in got:
        gb.close()


@pytest.mark.parametrize("graph", GRAPHS)
@pytest.mark.parametrize("settings", [dict(PG_EDGE=0, PG_SWEEP=0, PG_LIGHT=1), dict(PG_EDGE=0, PG_SWEEP=0, PG_LIGHT=0, PG_LAZY=1),
                                      dict(PG_EDGE=0, PG_SWEEP=1, PG_MIXED=0), dict(PG_EDGE=0, PG_SWEEP=1, PG_MIXED=1),
                                      dict(PG_EDGE=0, PG_SWEEP=1, PG_LIGHT=0, PG_LAZY=1), dict(PG_EDGE=1)], ids=str)
def test_bytes_of_a_run_are_those_of_its_launches(graph, settings):
    from paper_2008_01425_amd import binding as B
    from paper_2008_01425_amd.device import GossipBuffers
    for rank, steps in ((1, 1), (2, 2)):
        wl = _workload(graph, [(64, 96), (33, 130), (100, 1), (7, 8)] + ([(5, 12001)] if settings.get("PG_SWEEP") else []), rank, steps)
        print(f"case {wl.name} {settings}", flush=True)
        with env_settings(settings):
            gb = GossipBuffers.from_workload(wl)
        for rounds in (1, 2, 3, 4):
            B.pg_profile_enable(gb.ctx, True)
            gb.run(rounds)
            booked = sum(r["bytes"] for r in B.pg_profile_collect(gb.ctx))
            B.pg_profile_enable(gb.ctx, False)
            told = B.pg_run_bytes(gb.ctx, rounds)
            assert abs(booked - told) <= 1e-9 * told, (rank, steps, rounds, booked, told)
        gb.close()
