"""Passes of large parameter sets: streamed past the caches, and runs that write the parameters
every second round.  Both perform the operations of the plain passes on every element, so each is
held to the plain passes bit for bit (and those to the CPU oracle elsewhere)."""
import numpy as np
import pytest

from paper_2008_01425_amd import workloads as W
from parity_util import env_setting

pytestmark = pytest.mark.gpu

# every vector width, rows shorter and longer than a wavefront's step, several column segments, row
# counts around the eight rows of a lane group and the staged row blocks, vectors, single entries
SHAPES = [(64, 576), (33, 130), (17, 259), (5, 4609), (1030, 36), (9, 3), (700, 1), (1, 77), (1, 1), (7, 8), (8, 2306)]
TALL = SHAPES + [(4500, 33)]   # more than 4096 rows: Phat by the chunked kernels


def _workload(name, n, edges, rank, steps, sigma=0.05, shapes=SHAPES):
    edges = np.asarray(edges, np.int32).reshape(-1, 2)
    deg = np.bincount(edges.reshape(-1), minlength=n)
    w = np.array([1.0 / (1 + max(deg[a], deg[b])) for a, b in edges], np.float32)
    return W.Workload(name, n, edges, w, shapes, rank, steps, sigma, 10, 77)


def _buffers(wl, X, Q, stream, lazy, odd):
    """`odd`: whether the kernels that move rows of odd length four floats at a time are used.  The wide
    kernels' units are held fixed, so that `stream` changes nothing but the cache hint."""
    from paper_2008_01425_amd.device import GossipBuffers
    with env_setting("PG_STREAM", stream), env_setting("PG_LAZY", lazy), env_setting("PG_LIGHT", 0), \
            env_setting("PG_ODD_ROWS", odd), env_setting("PG_WIDE_UNITS", odd):
        gb = GossipBuffers.from_workload(wl, fill=False)
    gb.fill_from_arrays(X, Q)
    return gb


def _same(a, b, wl, what):
    from paper_2008_01425_amd import binding as B
    for i in range(wl.n_workers):
        assert bool((a.x[i].view(-1) == b.x[i].view(-1)).all()), (what, "worker", i)
    assert bool((a.q == b.q).all()), (what, "state")
    wa, wb = a.ws.view(-1), b.ws.view(-1)
    for l, (p, _) in enumerate(wl.shapes):
        r = wl.layer_rank(l)
        for e in range(wl.n_edges):
            for off, size in ((B.pg_ws_phat_offset(a.ctx, e, l), 4 * r * p), (B.pg_ws_flag_offset(a.ctx, e, l), 4 * r)):
                assert bool((wa[off:off + size] == wb[off:off + size]).all()), (what, "unit vectors or flags", e, l)


GRAPHS = {"ring": (4, [(0, 1), (1, 2), (2, 3), (3, 0)]),          # two (four) stacked columns everywhere
          "path": (4, [(1, 0), (1, 2), (3, 2)]),                  # one and two (two and four)
          "pair and a lone worker": (3, [(0, 1)])}
STARS = {"three columns": (5, [(0, 1), (2, 0), (0, 3)]),          # a kernel compiled for four; worker 4 alone
         "four columns": (5, [(0, 1), (2, 0), (0, 3), (4, 0)])}


def _run_profiled(gb, rounds):
    """gb.run(rounds), and what it launched: {kind: launches}.  The bytes booked are the run's."""
    from paper_2008_01425_amd import binding as B
    B.pg_profile_enable(gb.ctx, True)
    gb.run(rounds)
    rows = B.pg_profile_collect(gb.ctx)
    B.pg_profile_enable(gb.ctx, False)
    moved = B.pg_run_bytes(gb.ctx, rounds)
    assert abs(sum(r["bytes"] for r in rows) - moved) <= 1e-9 * moved
    return {r["name"]: r["launches"] for r in rows}


@pytest.mark.parametrize("graph", GRAPHS)
@pytest.mark.parametrize("rounds", [2, 3, 4, 7])
@pytest.mark.parametrize("rank", [1, 2])
@pytest.mark.parametrize("odd", [0, 1])
def test_a_run_that_writes_every_second_round_equals_the_plain_run(graph, rounds, rank, odd):
    _run_both(f"lazy {graph} {rounds} r{rank}", *GRAPHS[graph], rounds, rank, odd)


@pytest.mark.parametrize("graph", STARS)
@pytest.mark.parametrize("rounds", [2, 5])
@pytest.mark.parametrize("odd", [0, 1])
def test_a_run_that_writes_every_second_round_with_three_and_four_neighbours(graph, rounds, odd):
    _run_both(f"lazy star {graph} {rounds}", *STARS[graph], rounds, 1, odd)


def _run_both(name, n, edges, rounds, rank, odd):
    wl = _workload(name, n, edges, rank, 1, shapes=TALL)
    X, Q = wl.all_params(), wl.all_q()
    for l in (1, 6):                                   # two neighbours agree: their columns are dropped
        X[1][l] = X[0][l].copy()
    plain, lazy = _buffers(wl, X, Q, 0, 0, odd), _buffers(wl, X, Q, 1, 1, odd)
    for _ in range(2):                                 # the second call starts on what the first left
        did, did_lazily = _run_profiled(plain, rounds), _run_profiled(lazy, rounds)
        # no silent comparison of the plain run with itself
        assert "peek_sweep_p" not in did and did["update_sweep_p"] > 0
        assert did_lazily["peek_sweep_p"] > 0 and did_lazily["peek_sweep_q"] > 0
        assert ("update_sweep_p" in did_lazily) == (rounds > 2)
        _same(plain, lazy, wl, wl.name)
    plain.round()
    lazy.round()
    _same(plain, lazy, wl, wl.name + " and one round")
    plain.close()
    lazy.close()


@pytest.mark.parametrize("rank", [1, 2, 3, 4])
@pytest.mark.parametrize("odd", [0, 1])
def test_streamed_passes_equal_the_cached_ones(rank, odd):
    """1 to 16 stacked columns: every row and column kernel, each call."""
    import torch
    n, edges = 6, [(0, 1), (0, 2), (3, 0), (0, 4), (2, 1), (4, 5)]   # degrees 4, 2, 2, 1, 2, 1
    wl = _workload(f"stream r{rank}", n, edges, rank, 2)
    X, Q = wl.all_params(), wl.all_q()
    a, b = _buffers(wl, X, Q, 0, 0, odd), _buffers(wl, X, Q, 1, 1, odd)
    for gb in (a, b):
        gb.alloc_grads()
        gb.alloc_pstate()
        for i, g in enumerate(gb.g):
            g.normal_(generator=torch.Generator(device=g.device).manual_seed(i))
    for what, call in (("round", lambda gb: gb.round()), ("run", lambda gb: gb.run(3)),
                       ("sgd", lambda gb: gb.round_sgd(0.1)), ("odd iteration", lambda gb: gb.iterate(0, 1, 0.1)),
                       ("even iteration", lambda gb: gb.iterate(1, 1))):
        call(a)
        call(b)
        _same(a, b, wl, f"{wl.name} {what}")
    a.close()
    b.close()


@pytest.mark.parametrize("stream", [0, 1])
@pytest.mark.parametrize("rank", [2, 4])
def test_padding_of_rows_is_neither_used_nor_written(rank, stream):
    """Rows of 65, 66, 67 and more columns in a graph whose workers stack 2 to 16 columns: the wide kernels
    read such rows in units of four floats, the last of which reaches into the padding.  NaNs there
    stay where they are and change no result."""
    import torch
    from paper_2008_01425_amd.device import GossipBuffers
    edges = [(0, 1), (0, 2), (3, 0), (0, 4), (2, 1), (4, 5)]
    wl = _workload(f"padding r{rank}", 6, edges, rank, 1)
    shapes = [(40, 65), (33, 66), (70, 67), (129, 130), (17, 259), (9, 3277), (16, 1023), (300, 72)]
    wl = W.Workload(wl.name, 6, wl.edges, wl.edge_w, shapes, rank, 1, 0.05, 10, 78)
    X, Q = wl.all_params(), wl.all_q()
    bufs = []
    for pad in (0.0, float("nan")):
        with env_setting("PG_STREAM", stream), env_setting("PG_LIGHT", 0):
            gb = GossipBuffers.from_workload(wl, fill=False)
        gb.alloc_grads()
        gb.alloc_pstate()
        for i in range(gb.n):
            gb.x[i].fill_(pad)
            gb.g[i].fill_(pad)
        gb.fill_from_arrays(X, Q)
        for i in range(gb.n):
            for l, s in enumerate(shapes):
                gb.set_grad_layer(i, l, X[i][l][::-1] * 0.1)
        bufs.append(gb)
    a, b = bufs
    holes = [torch.isnan(x) for x in b.x]
    assert all(int(h.sum()) > 0 for h in holes)
    for what, call in (("round", lambda gb: gb.round()), ("run", lambda gb: gb.run(3)),
                       ("sgd", lambda gb: gb.round_sgd(0.1)), ("odd iteration", lambda gb: gb.iterate(0, 1, 0.1)),
                       ("even iteration", lambda gb: gb.iterate(1, 1, 0.1))):
        for gb in bufs:
            call(gb)
        for i in range(a.n):
            assert bool((torch.isnan(b.x[i]) == holes[i]).all()), (what, i)
            assert bool((torch.nan_to_num(b.x[i]) == a.x[i]).all()), (what, i)
            assert bool((a.x[i][holes[i]] == 0).all()), (what, i)
        assert bool((a.q == b.q).all()) and bool((a.pstate == b.pstate).all()), what
    for gb in bufs:
        gb.close()


def _against_the_oracle(name, shapes, rank, seed, light, odd, steps=1, graph="ring"):
    """A round, a round with gradient, an odd and an even iteration on `shapes`; the one-round bar of the
    other parity tests."""
    from oracle import pg_oracle as O
    from parity_util import TOL_1, compare_state, oracle_problem
    from paper_2008_01425_amd.device import GossipBuffers
    n, edges = GRAPHS[graph]
    wl = _workload(name, n, edges, rank, steps)
    wl = W.Workload(f"{name} r{rank}", n, wl.edges, wl.edge_w, shapes, rank, steps, 0.05, 10, seed)
    layers = list(range(len(shapes)))
    prob, eta = oracle_problem(wl), 0.05
    rng = np.random.default_rng(5)
    G = [[rng.standard_normal(s).astype(np.float32) for s in shapes] for _ in range(n)]
    for what in ("round", "sgd", "iterations"):
        X, Q = wl.all_params(), wl.all_q()
        with env_setting("PG_LIGHT", light), env_setting("PG_ODD_ROWS", odd):
            gb = GossipBuffers.from_workload(wl, fill=False)
        gb.fill_from_arrays(X, Q)
        gb.alloc_grads()
        gb.alloc_pstate()
        for i in range(n):
            for l in layers:
                gb.set_grad_layer(i, l, G[i][l])
        if what == "round":
            gb.round()
            O.gossip_round(prob, X, Q)
        elif what == "sgd":
            gb.round_sgd(eta)
            O.gossip_round(prob, X, Q, G=G, eta=float(np.float32(eta)))
        else:
            P = [[np.zeros((wl.layer_rank(l), shapes[l][0]), np.float32) for l in layers] for _ in range(wl.n_edges)]
            gb.iterate(0, 2, eta)
            O.alg2_round(prob, X, Q, P, 0, 2, G=G, eta=float(np.float32(eta)))
        print(f"   {what}: worst rel err", compare_state(gb, X, Q, layers, TOL_1, what=f"{wl.name} {what}"), flush=True)
        gb.close()


@pytest.mark.parametrize("rank", [1, 2])
@pytest.mark.parametrize("light", [0, 1])
@pytest.mark.parametrize("odd", [0, 1])
def test_rows_of_any_length_and_alignment(rank, light, odd):
    """Rows of 16 and more floats at any 4-byte aligned address (every remainder modulo 4; a last unit
    that overlaps its neighbour's, alone in a row or behind many), in units of four and in the widths that
    divide the row, against the oracle: a round, a round with gradient, an odd and an even iteration."""
    shapes = [(9, 17), (40, 18), (33, 19), (21, 16), (70, 255), (130, 257), (20, 1022), (65, 1023), (6, 4099)]
    _against_the_oracle("any alignment", shapes, rank, 79, light, odd)


@pytest.mark.parametrize("rank", [1, 2])
@pytest.mark.parametrize("light", [0, 1])
@pytest.mark.parametrize("odd", [0, 1])
def test_rows_shorter_than_sixteen_floats(rank, light, odd):
    """Two floats at a time where q is even, one at a time where it is odd: q = 2 to 15, several row blocks
    and fewer rows than a lane group takes."""
    shapes = [(50, 2), (7, 6), (1030, 10), (33, 14), (260, 5), (9, 15), (3000, 6), (40, 3), (2, 14), (70, 12)]
    _against_the_oracle("short rows", shapes, rank, 80, light, odd)
