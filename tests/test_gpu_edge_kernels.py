"""Sets of small layers: one work-group per (edge, layer) between two updates, against the oracle and, call
by call, against the streaming kernels."""
import numpy as np
import pytest

from oracle import pg_oracle as O
from parity_util import TOL_1, TOL_10, compare_state, env_setting, graph_workload, launched, oracle_problem, oracle_rounds

pytestmark = pytest.mark.gpu

# thread splits of a work-group: one row per thread and one unit, rows over many wavefronts, all threads rows, all units used,
# every remainder of q modulo 4, row counts around powers of two, vectors, single entries
SHAPES = {
    256: [(64, 32), (32, 16), (16, 1), (1, 1), (1, 9), (3, 3000), (256, 36), (255, 33), (17, 259), (65, 70), (9, 3), (33, 130), (250, 1)],
    512: [(32, 576), (100, 100), (512, 36), (500, 1), (257, 30), (8, 1540), (1, 5000), (2, 4001), (5, 1601), (129, 66), (77, 101)],
}
GRAPHS = {"ring": (5, [(0, 1), (1, 2), (2, 3), (3, 4), (4, 0)]),
          "hub, leaves and a lone worker": (7, [(0, 1), (2, 0), (0, 3), (4, 0), (3, 5)])}


def _workload(graph, shapes, rank, steps, seed=31):
    return graph_workload(f"edge {graph} {len(shapes)} r{rank}", GRAPHS[graph], shapes, rank, steps, seed)


def _buffers(wl, X, Q, edge):
    from paper_2008_01425_amd.device import GossipBuffers
    with env_setting("PG_EDGE", edge):
        gb = GossipBuffers.from_workload(wl, fill=False)
    gb.fill_from_arrays(X, Q)
    return gb


@pytest.mark.parametrize("threads", SHAPES)
@pytest.mark.parametrize("graph", GRAPHS)
@pytest.mark.parametrize("rank,steps", [(1, 1), (2, 2), (3, 1), (4, 1)])
def test_rounds_runs_and_gradients_against_the_oracle(threads, graph, rank, steps):
    wl = _workload(graph, SHAPES[threads], rank, steps)
    layers = list(range(len(wl.shapes)))
    prob = oracle_problem(wl)
    X, Q = wl.all_params(), wl.all_q()
    for l in (0, 2):                                  # two neighbours agree: their columns are dropped
        X[1][l] = X[0][l].copy()
    print(f"case {wl.name} {threads}", flush=True)
    a, b, c, d = (_buffers(wl, X, Q, 1) for _ in range(4))
    kinds = launched(a, a.round)
    assert kinds == {"edge": 1, "update": 1}, kinds
    kinds = launched(b, lambda: b.run(3))
    # one launch a round where the operands of a pending update fit beside each other, at high ranks two
    assert kinds["edge"] == 3 and kinds["update"] in ((1,) if graph == "ring" and rank == 1 else (1, 3)), kinds
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
    compare_state(b, snaps[3].X, snaps[3].Q, layers, TOL_10, what="run of 3", phat=snaps[3].phat, flags=snaps[3].degenerate)
    compare_state(c, X, Q, layers, TOL_10, what="run of 4", phat=info.phat, flags=info.degenerate)
    for _ in range(3):                                # a run is its rounds, bit for bit
        a.round()
    assert all(bool((x == y).all()) for x, y in zip(a.x, c.x)) and bool((a.q == c.q).all())
    for gb in (a, b, c, d):
        gb.close()


@pytest.mark.parametrize("threads", SHAPES)
@pytest.mark.parametrize("rank", [1, 2, 4])
def test_single_iterations_against_the_oracle(threads, rank):
    wl = _workload("hub, leaves and a lone worker", SHAPES[threads], rank, 1, 32)
    layers = list(range(len(wl.shapes)))
    prob, eta = oracle_problem(wl), 0.05
    rng = np.random.default_rng(6)
    X, Q = wl.all_params(), wl.all_q()
    X[1][0] = X[0][0].copy()
    P = [[np.zeros((wl.layer_rank(l), wl.shapes[l][0]), np.float32) for l in layers] for _ in range(wl.n_edges)]
    gb = _buffers(wl, X, Q, 1)
    gb.alloc_pstate()
    gb.alloc_grads()
    print(f"case iterate {wl.name} {threads}", flush=True)
    done = 0
    for its, grad in ((1, True), (1, False), (2, True), (3, False), (2, True)):
        G = None
        if grad:
            G = [[rng.standard_normal(s).astype(np.float32) for s in wl.shapes] for _ in range(wl.n_workers)]
            for i in range(wl.n_workers):
                for l in layers:
                    gb.set_grad_layer(i, l, G[i][l])
        gb.iterate(done, its, eta if grad else None)
        drop = O.alg2_round(prob, X, Q, P, done, its, G=G, eta=float(np.float32(eta)) if grad else 0.0)
        done += its
        compare_state(gb, X, Q, layers, TOL_1 if done == 1 else TOL_10, what=f"iterations to {done}", flags=drop)
    from parity_util import rel_err
    for l in layers:
        for e in range(wl.n_edges):
            assert rel_err(gb.get_p(e, l), P[e][l]) <= TOL_10
    gb.close()


def test_a_layer_that_does_not_fit_keeps_the_set_on_the_streaming_kernels():
    for shapes in ([(64, 32), (513, 4)], [(64, 32), (33, 576)], [(64, 32), (1, 18433)]):
        wl = _workload("ring", shapes, 1, 1)
        gb = _buffers(wl, wl.all_params(), wl.all_q(), 1)
        assert "edge" not in launched(gb, gb.round), shapes
        gb.close()


@pytest.mark.parametrize("rounds", [2, 3])
def test_runs_with_sixteen_columns_are_their_rounds(rounds):
    """More than eight columns: the update in fours of columns, at a run's end from the second buffer (even) or in place."""
    wl = _workload("hub, leaves and a lone worker", [(33, 40), (20, 64), (64, 1), (7, 9), (1, 77)], 4, 1, 33)
    X, Q = wl.all_params(), wl.all_q()
    layers = list(range(len(wl.shapes)))
    print(f"case {wl.name} {rounds}", flush=True)
    a, b = _buffers(wl, X, Q, 1), _buffers(wl, X, Q, 1)
    assert launched(a, lambda: a.run(rounds)) == {"edge": rounds, "update": 1}
    for _ in range(rounds):
        b.round()
    assert all(bool((x == y).all()) for x, y in zip(a.x, b.x)) and bool((a.q == b.q).all())
    info = oracle_rounds(wl, X, Q, rounds, layers)
    compare_state(a, X, Q, layers, TOL_10, what=f"run of {rounds}", flags=info.degenerate)
    a.close()
    b.close()
