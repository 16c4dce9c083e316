"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element by element,
on the same seeded inputs.  Tolerances: 1e-5 relative per element after one round, 1e-4 after
ten (rel_err in parity_util: |g - o| / max(|o|, rms(o)))."""
import numpy as np
import pytest

from paper_2008_01425_amd import workloads as W
import os
import time

from parity_util import PATHS, TOL_1, TOL_10, compare_state, env_settings, launched, oracle_rounds, rel_err

pytestmark = pytest.mark.gpu


def _gb(wl, layers=None, arrays=None):
    """Device buffers of a workload, filled from the seeded generator or from (X, Q) host arrays
    already drawn from it."""
    from paper_2008_01425_amd.device import GossipBuffers
    gb = GossipBuffers.from_workload(wl, fill=False)
    if arrays is None:
        gb.fill_from_workload(wl, layers)
    else:
        gb.fill_from_arrays(arrays[0], arrays[1], layers)
    return gb


def _custom(name, n, edges, w, shapes, rank, steps, sigma=0.05, seed=1):
    ew = np.full((len(edges),), w, dtype=np.float32) if np.isscalar(w) else np.asarray(w, np.float32)
    return W.Workload(name, n, np.asarray(edges, dtype=np.int32).reshape(-1, 2), ew, shapes, rank,
                      steps, sigma, 10, seed)


def _check(wl, rounds, tol, fused=False, layers=None, two_calls=False):
    layers = list(range(len(wl.shapes))) if layers is None else list(layers)
    print(f"case {wl.name} rounds={rounds} fused={fused} layers={layers[:6]}", flush=True)
    X, Q = wl.all_params(layers), wl.all_q(layers)
    gb = _gb(wl, layers, (X, Q))
    if fused:
        if two_calls:
            gb.run(rounds - rounds // 2)
            gb.run(rounds // 2)
        else:
            gb.run(rounds)
    else:
        for _ in range(rounds):
            gb.round()
    info = oracle_rounds(wl, X, Q, rounds, layers)
    worst = compare_state(gb, X, Q, layers, tol, what=wl.name, phat=info.phat, flags=info.degenerate)
    print("   worst rel err", worst, flush=True)
    gb.close()
    return worst


def _check_named(name, rounds=10):
    """A named configuration at full size, every layer: one oracle trajectory of `rounds` rounds
    (snapshot after the first) against (a) one pg_round call at the one-round tolerance, (b) that
    context continued by single pg_round calls, (c) one pg_run(rounds) on a second context, both
    at the ten-round tolerance.  Parameters, state, orthonormal columns and dropped flags."""
    wl = W.get(name)
    layers = list(range(len(wl.shapes)))
    t0 = time.time()
    X, Q = wl.all_params(), wl.all_q()
    print(f"case {name} all {len(layers)} layers: inputs drawn {time.time() - t0:.0f} s", flush=True)
    a = _gb(wl, layers, (X, Q))
    b = _gb(wl, layers, (X, Q))
    a.round()
    b.run(rounds)
    print(f"   device buffers filled, first GPU rounds queued {time.time() - t0:.0f} s", flush=True)
    info, snaps = oracle_rounds(wl, X, Q, rounds, layers, snap_at=(1,))
    print(f"   oracle: {rounds} rounds {time.time() - t0:.0f} s", flush=True)
    s1 = snaps[1]
    w1 = compare_state(a, s1.X, s1.Q, layers, TOL_1, what=name + " round 1", phat=s1.phat, flags=s1.degenerate)
    print("   1 round (pg_round)      worst rel err", w1, flush=True)
    del snaps, s1
    for _ in range(rounds - 1):
        a.round()
    w2 = compare_state(a, X, Q, layers, TOL_10, what=f"{name} {rounds} x pg_round", phat=info.phat, flags=info.degenerate)
    print(f"   {rounds} x pg_round          worst rel err", w2, flush=True)
    a.close()
    w3 = compare_state(b, X, Q, layers, TOL_10, what=f"{name} pg_run({rounds})", phat=info.phat, flags=info.degenerate)
    print(f"   pg_run({rounds})              worst rel err", w3, f"{time.time() - t0:.0f} s", flush=True)
    b.close()


# ------------------------------------------------------------------ the named configurations
def test_tiny_one_round():
    _check(W.get("tiny"), 1, TOL_1)


def test_tiny_ten_rounds():
    _check(W.get("tiny"), 10, TOL_10)


def test_tiny_ten_rounds_fused_run():
    _check(W.get("tiny"), 10, TOL_10, fused=True)


def test_resnet20_one_round_and_ten():
    _check(W.get("resnet20"), 1, TOL_1)
    _check(W.get("resnet20"), 10, TOL_10, fused=True)


# ------------------------------------------------------------------ shapes, ranks, topologies
SHAPES_RAGGED = [(37, 27), (130, 50), (9, 147), (300, 260), (700, 1), (5, 3), (1, 8), (64, 1028)]


@pytest.mark.parametrize("rank,steps", [(1, 1), (2, 1), (4, 2), (3, 1)])
def test_ragged_shapes_ring(rank, steps):
    wl = _custom(f"ragged_r{rank}s{steps}", 5, W.ring_edges(5), 1 / 3, SHAPES_RAGGED, rank, steps)
    _check(wl, 1, TOL_1)
    _check(wl, 3, TOL_10, fused=True, two_calls=True)


def test_torus_rank4_two_steps():
    wl = _custom("torus3x3", 9, W.torus_edges(3, 3), 1 / 5, [(200, 650), (33, 12), (40, 1)], 4, 2)
    _check(wl, 1, TOL_1)
    _check(wl, 4, TOL_10, fused=True)


def test_irregular_graph_with_isolated_and_leaf_workers():
    edges = [[0, 1], [2, 0], [0, 3], [3, 1]]          # worker 4 has no edge; degrees 3, 2, 1, 2, 0
    wl = _custom("irregular", 5, edges, [0.3, 0.2, 0.25, 0.4], [(48, 36), (17, 1), (20, 64)], 2, 1)
    _check(wl, 2, TOL_10)
    _check(wl, 2, TOL_10, fused=True)


def test_sixteen_stacked_columns_mixed_degrees_and_odd_shapes():
    """Rank 4 on a star with a chord: workers with 16, 8, 8, 4 and 4 stacked columns share every
    layer (matrix-core and vector kernels side by side); odd, short and just-over-a-step row
    lengths, row counts around the 16-row blocks."""
    edges = [[0, 1], [0, 2], [3, 0], [0, 4], [2, 1]]
    shapes = [(50, 131), (17, 70), (100, 64), (9, 3), (33, 200), (16, 65), (1, 40)]
    wl = _custom("star16", 5, edges, [0.2, 0.2, 0.2, 0.2, 0.15], shapes, 4, 2)
    _check(wl, 1, TOL_1)
    _check(wl, 3, TOL_10, fused=True)
    wl = _custom("star16_sgd", 5, edges, [0.2, 0.2, 0.2, 0.2, 0.15], shapes, 4, 1)
    _check_sgd(wl, [0.1, 0.05], TOL_10)


@pytest.mark.parametrize("n,edges,w,rank", [
    (2, [[0, 1]], 0.3, 16),                 # one edge at the largest rank: column-by-column Gram-Schmidt
    (3, [[0, 1], [1, 2]], 0.4, 8),          # path: 8, 16 and 8 stacked columns
    (3, [[0, 1], [2, 1]], 0.3, 6),          # ranks between the compiled sizes
])
def test_high_ranks(n, edges, w, rank):
    shapes = [(70, 90), (40, 200), (24, 17), (12, 300), (5, 64)]
    wl = _custom(f"rank{rank}_n{n}", n, edges, w, shapes, rank, 2, sigma=0.1)
    _check(wl, 1, TOL_1)
    _check(wl, 3, TOL_10, fused=True)


def test_many_tiles_and_tail_rows():
    wl = _custom("tall", 3, W.ring_edges(3), 1 / 3, [(4099, 68), (1031, 516), (70, 4612)], 2, 1)
    _check(wl, 1, TOL_1)
    _check(wl, 2, TOL_10, fused=True)


def test_tall_embedding_shaped_layer():
    """33278 x 650: rows only 8-byte aligned, row chunks in the orthonormalisation, many row blocks."""
    wl = _custom("tall_embedding", 3, W.ring_edges(3), 1 / 3, [(33278, 650)], 2, 2, sigma=0.01)
    _check(wl, 1, TOL_1)
    _check(wl, 2, TOL_10, fused=True)
    # single iterations: the vectors in R^p are normalised and combined chunk by chunk as well
    wl = _custom("tall_embedding_iter", 3, W.ring_edges(3), 1 / 3, [(33278, 650), (5000, 1), (40, 30)], 2, 1, sigma=0.01)
    _check_iterate(wl, [1, 1, 1, 1], TOL_10, eta=0.05)


def test_random_projections_fresh_state_every_round():
    """Section 5, 'Random projections vs. power iteration': the same round with a fresh N(0,1)
    projection every time instead of the warm start -- the caller simply refills the state.
    The paper's consensus setting: 8-ring, W_ij = 0.436, 100 x 100 standard normal matrices."""
    from paper_2008_01425_amd.device import GossipBuffers
    from parity_util import oracle_problem
    from oracle import pg_oracle as O
    n = 8
    wl = W.Workload("consensus_gauss", n, W.ring_edges(n), np.full((n,), 0.436, np.float32),
                    [(100, 100)], 1, 1, 1.0, 10, 7)
    rng = np.random.default_rng(123)
    X = [[rng.standard_normal((100, 100)).astype(np.float32)] for _ in range(n)]
    gb = GossipBuffers.from_workload(wl, fill=False)
    for i in range(n):
        gb.set_layer(i, 0, X[i][0])
    prob = oracle_problem(wl)
    for t in range(5):
        Q = [[rng.standard_normal((1, 100)).astype(np.float32)] for _ in range(n)]
        for e in range(n):
            gb.set_q(e, 0, Q[e][0])
        gb.round()
        O.gossip_round(prob, X, Q)
    for i in range(n):
        assert rel_err(gb.get_layer(i, 0), X[i][0]) <= TOL_10
    gb.close()


# ------------------------------------------------------------------ Algorithm 1: fused gradient term
def _check_sgd(wl, steps_eta, tol):
    """pg_round_sgd against the oracle's Algorithm-1 step, fresh random gradients every step."""
    from oracle import pg_oracle as O
    from parity_util import oracle_problem
    print(f"case sgd {wl.name}", flush=True)
    gb = _gb(wl)
    gb.alloc_grads()
    layers = list(range(len(wl.shapes)))
    X, Q = wl.all_params(), wl.all_q()
    prob = oracle_problem(wl)
    rng = np.random.default_rng(99)
    for eta in steps_eta:
        G = [[rng.standard_normal(s).astype(np.float32) for s in wl.shapes] for _ in range(wl.n_workers)]
        for i in range(wl.n_workers):
            for l in layers:
                gb.set_grad_layer(i, l, G[i][l])
        gb.round_sgd(eta)
        O.gossip_round(prob, X, Q, G=G, eta=float(np.float32(eta)))
    worst = compare_state(gb, X, Q, layers, tol, what="sgd " + wl.name)
    print("   worst rel err", worst, flush=True)
    gb.close()


@pytest.mark.parametrize("rank,steps", [(1, 1), (2, 2), (4, 1)])
def test_sgd_step_ragged_ring(rank, steps):
    wl = _custom(f"sgd_ragged_r{rank}", 5, W.ring_edges(5), 1 / 3, SHAPES_RAGGED, rank, steps)
    _check_sgd(wl, [0.1], TOL_1)
    _check_sgd(wl, [0.05, 0.02, 0.01], TOL_10)


def test_sgd_step_torus_sixteen_columns_and_isolated_worker():
    wl = _custom("sgd_torus", 9, W.torus_edges(3, 3), 1 / 5, [(200, 650), (33, 12), (40, 1)], 4, 1)
    _check_sgd(wl, [0.1, 0.1], TOL_10)
    edges = [[0, 1], [2, 0], [0, 3], [3, 1]]          # worker 4 has no edge: plain SGD for it
    wl = _custom("sgd_irregular", 5, edges, [0.3, 0.2, 0.25, 0.4], [(48, 36), (17, 1), (20, 64)], 2, 1)
    _check_sgd(wl, [0.1, 0.2], TOL_10)


def test_sgd_step_without_any_edge_is_plain_sgd():
    from paper_2008_01425_amd.device import GossipBuffers
    gb = GossipBuffers(2, np.zeros((0, 2), np.int32), np.zeros((0,), np.float32), [(8, 4), (5, 1)], 1, 1)
    gb.alloc_grads()
    rng = np.random.default_rng(3)
    xs = [[rng.standard_normal(s).astype(np.float32) for s in gb.shapes] for _ in range(2)]
    gs = [[rng.standard_normal(s).astype(np.float32) for s in gb.shapes] for _ in range(2)]
    for i in range(2):
        for l in range(2):
            gb.set_layer(i, l, xs[i][l]); gb.set_grad_layer(i, l, gs[i][l])
    gb.round_sgd(0.25)
    for i in range(2):
        for l in range(2):
            want = (xs[i][l].astype(np.float64) - 0.25 * gs[i][l].astype(np.float64)).astype(np.float32)
            assert np.array_equal(gb.get_layer(i, l), want)
    gb.close()


def test_sgd_step_vgg16_full_size_sampled_layers():
    wl = W.get("vgg16_r1")
    from oracle import pg_oracle as O
    from parity_util import oracle_rounds
    layers = [0, 5, 13]
    gb = _gb(wl, layers)
    gb.alloc_grads()
    X, Q = wl.all_params(layers), wl.all_q(layers)
    rng = np.random.default_rng(5)
    G = [[rng.standard_normal(wl.shapes[l]).astype(np.float32) for l in layers] for _ in range(wl.n_workers)]
    for i in range(wl.n_workers):
        for j, l in enumerate(layers):
            gb.set_grad_layer(i, l, G[i][j])
    gb.round_sgd(0.01)
    sub = O.Problem(wl.n_workers, wl.edges, wl.edge_w.astype(np.float64), [wl.shapes[l] for l in layers], 1, 1)
    O.gossip_round(sub, X, Q, G=G, eta=float(np.float32(0.01)))
    compare_state(gb, X, Q, layers, TOL_1, what="sgd vgg16")
    gb.close()


# ------------------------------------------------------------------ Algorithm 2, one iteration at a time
def _check_iterate(wl, schedule, tol, eta=None):
    """pg_iterate against the oracle's literal Algorithm 2 over a schedule of iteration counts."""
    from oracle import pg_oracle as O
    from parity_util import oracle_problem
    print(f"case iterate {wl.name} schedule={schedule} eta={eta}", flush=True)
    gb = _gb(wl)
    gb.alloc_pstate()
    if eta is not None:
        gb.alloc_grads()
    L, E = len(wl.shapes), wl.n_edges
    X, Vq = wl.all_params(), wl.all_q()
    Vp = [[np.zeros((wl.layer_rank(l), wl.shapes[l][0]), np.float32) for l in range(L)] for _ in range(E)]
    prob = oracle_problem(wl)
    rng = np.random.default_rng(17)
    k = 0
    for its in schedule:
        G = None
        if eta is not None:
            G = [[rng.standard_normal(s).astype(np.float32) for s in wl.shapes] for _ in range(wl.n_workers)]
            for i in range(wl.n_workers):
                for l in range(L):
                    gb.set_grad_layer(i, l, G[i][l])
        gb.iterate(k, its, eta)
        drop = O.alg2_round(prob, X, Vq, Vp, k, its, G=G, eta=0.0 if eta is None else float(np.float32(eta)))
        k += its
    worst = compare_state(gb, X, Vq, list(range(L)), tol, what="iterate " + wl.name, flags=drop)
    for l in range(L):
        for e in range(E):
            err = rel_err(gb.get_p(e, l), Vp[e][l])
            worst["ph"] = max(worst["ph"], err)
            assert err <= tol, f"p-state edge {e} layer {l}: {err:.3e}"
    print("   worst rel err", worst, flush=True)
    gb.close()


@pytest.mark.parametrize("rank", [1, 2, 4])
def test_single_iterations_ragged_ring(rank):
    wl = _custom(f"iter_ragged_r{rank}", 5, W.ring_edges(5), 1 / 3, SHAPES_RAGGED, rank, 1)
    _check_iterate(wl, [1], TOL_1)
    _check_iterate(wl, [1, 1, 1, 1], TOL_10)
    _check_iterate(wl, [2, 3, 1, 2], TOL_10)


def test_single_iterations_with_gradients_on_a_torus():
    wl = _custom("iter_torus", 9, W.torus_edges(3, 3), 1 / 5, [(120, 260), (33, 12), (40, 1)], 2, 1)
    _check_iterate(wl, [1, 1, 2], TOL_10, eta=0.05)
    # rank 4: 16 stacked columns (matrix-core row and column passes on the alternate buffers)
    wl = _custom("iter_torus_r4", 9, W.torus_edges(3, 3), 1 / 5, [(120, 262), (33, 12), (40, 1)], 4, 1)
    _check_iterate(wl, [1, 1, 2], TOL_10, eta=0.05)
    _check_iterate(wl, [1, 1], TOL_10)


def test_two_iterations_match_one_power_step_on_the_gpu():
    """The paper's 'PowerGossip (2 iterations)' = one pg_round power step (same approximation)."""
    wl = W.get("resnet20")
    a, b = _gb(wl), _gb(wl)
    b.alloc_pstate()
    a.round()
    b.iterate(0, 2)
    for i in range(wl.n_workers):
        for l in range(len(wl.shapes)):
            assert rel_err(b.get_layer(i, l), a.get_layer(i, l)) <= TOL_1
    for e in range(wl.n_edges):
        for l in range(len(wl.shapes)):
            assert rel_err(b.get_q(e, l), a.get_q(e, l)) <= TOL_1
    a.close(); b.close()


def test_single_iteration_vgg16_full_size_sampled_layers():
    wl = W.get("vgg16_r1")
    from oracle import pg_oracle as O
    layers = [0, 5, 13]
    gb = _gb(wl, layers)
    gb.alloc_pstate()
    X, Vq = wl.all_params(layers), wl.all_q(layers)
    Vp = [[np.zeros((1, wl.shapes[l][0]), np.float32) for l in layers] for _ in range(wl.n_edges)]
    sub = O.Problem(wl.n_workers, wl.edges, wl.edge_w.astype(np.float64), [wl.shapes[l] for l in layers], 1, 1)
    k = 0
    for its in (1, 1, 1):
        gb.iterate(k, its)
        O.alg2_round(sub, X, Vq, Vp, k, its)
        k += its
    compare_state(gb, X, Vq, layers, TOL_10, what="iterate vgg16")
    for j, l in enumerate(layers):
        for e in range(wl.n_edges):
            assert rel_err(gb.get_p(e, l), Vp[e][j]) <= TOL_10
    gb.close()


# ------------------------------------------------------------------ degenerate cases
def test_identical_workers_are_a_fixed_point():
    from paper_2008_01425_amd.device import GossipBuffers
    wl = _custom("same", 4, W.ring_edges(4), 1 / 3, [(40, 24), (12, 1)], 2, 2, sigma=0.0)
    gb = GossipBuffers.from_workload(wl)
    x0 = [[gb.get_layer(i, l) for l in range(2)] for i in range(4)]
    q0 = [[gb.get_q(e, l) for l in range(2)] for e in range(4)]
    gb.run(3)
    gb.round()
    for i in range(4):
        for l in range(2):
            assert np.array_equal(gb.get_layer(i, l), x0[i][l])
    for e in range(4):
        for l in range(2):
            assert np.array_equal(gb.get_q(e, l), q0[e][l])
            assert gb.get_flags(e, l).all()
            assert not gb.get_phat(e, l).any()
    gb.close()


def test_rank_deficient_difference_drops_a_column():
    from paper_2008_01425_amd.device import GossipBuffers
    from oracle import pg_oracle as O
    rng = np.random.default_rng(5)
    p, q = 48, 40
    base = rng.standard_normal((p, q)).astype(np.float32)
    # a difference that is exactly rank one in float: small-integer outer product
    u = rng.integers(-3, 4, p).astype(np.float32)
    v = rng.integers(-3, 4, q).astype(np.float32)
    base = np.round(base * 64) / 64
    Xa, Xb = (base + np.outer(u, v) / 64).astype(np.float32), base.copy()
    Q0 = rng.standard_normal((2, q)).astype(np.float32)
    gb = GossipBuffers(2, [[0, 1]], [0.5], [(p, q)], 2, 1)
    gb.set_layer(0, 0, Xa); gb.set_layer(1, 0, Xb); gb.set_q(0, 0, Q0)
    gb.round()
    prob = O.Problem(2, np.array([[0, 1]]), np.array([0.5]), [(p, q)], 2, 1)
    X, Q = [[Xa.copy()], [Xb.copy()]], [[Q0.copy()]]
    info = O.gossip_round(prob, X, Q, want_phat=True)
    assert info.degenerate[0].tolist() == [[0, 1]]
    assert gb.get_flags(0, 0).tolist() == [0, 1]
    assert np.array_equal(gb.get_q(0, 0)[1], Q0[1])
    assert rel_err(gb.get_q(0, 0)[0], Q[0][0][0]) <= TOL_1
    assert rel_err(gb.get_layer(0, 0), X[0][0]) <= TOL_1
    assert rel_err(gb.get_layer(1, 0), X[1][0]) <= TOL_1
    gb.close()


def test_no_edges_is_a_no_op():
    from paper_2008_01425_amd.device import GossipBuffers
    gb = GossipBuffers(2, np.zeros((0, 2), np.int32), np.zeros((0,), np.float32), [(8, 4)], 1, 1)
    a = np.arange(32, dtype=np.float32).reshape(8, 4)
    gb.set_layer(0, 0, a)
    gb.round(); gb.run(2)
    assert np.array_equal(gb.get_layer(0, 0), a)
    gb.close()


def test_results_are_deterministic():
    wl = W.get("resnet20")
    outs = []
    for _ in range(2):
        gb = _gb(wl)
        gb.run(3)
        outs.append((gb.x[3].cpu().numpy().copy(), gb.q.cpu().numpy().copy()))
        gb.close()
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])


def test_run_equals_repeated_round_bitwise():
    wl = _custom("fuse_eq", 6, W.ring_edges(6), 1 / 3, [(96, 260), (50, 1), (31, 27)], 2, 2)
    a, b = _gb(wl), _gb(wl)
    a.run(4)
    for _ in range(4):
        b.round()
    for i in range(6):
        assert np.array_equal(a.x[i].cpu().numpy(), b.x[i].cpu().numpy())
    assert np.array_equal(a.q.cpu().numpy(), b.q.cpu().numpy())
    a.close(); b.close()


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("rank,steps", [(1, 1), (2, 2)])
def test_run_equals_repeated_round_bitwise_on_every_path(path, rank, steps):
    """On the streaming kernels a run shares a pass between an update and the next product, on edge kernels it applies
    an update in the next round's launch; edge sweeps run their rounds."""
    wl = _custom("fuse_eq", 6, W.ring_edges(6), 1 / 3, [(60, 90) if path == "edge kernels" else (96, 260), (50, 1), (31, 27)], rank, steps)
    with env_settings(PATHS[path]):
        a, b = _gb(wl), _gb(wl)
    print(f"case {path} rank {rank}", flush=True)
    run, rounds = launched(a, lambda: a.run(4)), launched(b, lambda: [b.round() for _ in range(4)])
    if path == "streaming kernels":
        assert run["update_sweep_p"] > 0 and "update_sweep_p" not in rounds, (run, rounds)
    elif path == "edge kernels":
        assert run == {"edge": 4, "update": 1} and rounds == {"edge": 4, "update": 4}, (run, rounds)
    else:
        assert run == rounds and run["edge_sweep"] == 4 * steps, (run, rounds)
    for i in range(6):
        assert np.array_equal(a.x[i].cpu().numpy(), b.x[i].cpu().numpy())
    assert np.array_equal(a.q.cpu().numpy(), b.q.cpu().numpy())
    a.close(); b.close()


def test_run_can_be_captured_in_a_graph_and_replayed():
    """After its first call pg_run only launches kernels, so a caller may capture it in a HIP
    graph.  Every replay (with eager work and synchronisation in between) must leave exactly
    what the same number of eager rounds leaves."""
    import torch
    wl = _custom("graph", 9, W.torus_edges(3, 3), 1 / 5, [(96, 260), (50, 1), (31, 27), (40, 130)], 2, 2)
    eager, cap = _gb(wl), _gb(wl)
    cap.run(1)          # first call: uploads the pointer table (not capturable), then rounds
    eager.run(1)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        cap.run(3)
    torch.cuda.synchronize()
    scratch = torch.zeros(1 << 20, device="cuda")
    for rep in range(4):                    # the capture itself executed nothing
        g.replay()
        eager.run(3)
        torch.cuda.synchronize()
        for i in range(9):
            assert np.array_equal(cap.x[i].cpu().numpy(), eager.x[i].cpu().numpy()), f"replay {rep}, worker {i}"
        assert np.array_equal(cap.q.cpu().numpy(), eager.q.cpu().numpy()), f"replay {rep}, state"
        scratch.add_(1.0).sum().item()      # unrelated eager work and a synchronisation between replays
    eager.close(); cap.close()


# ------------------------------------------------------------------ more than 16 stacked columns
def test_full_rank_on_the_gpu_is_plain_gossip():
    """r >= p <= q: Phat Phat^T is the identity and the round is X <- W X (Eq. (1) without the
    gradient; delta = 1 in Theorem 1).  On the 3 x 3 torus at rank 16 every worker has 24-64
    stacked columns, taken in groups of whole edges.  Against the oracle and against the dense
    product with the mixing matrix."""
    n, w = 9, 1 / 5
    edges = W.torus_edges(3, 3)
    shapes = [(6, 40), (12, 30), (16, 20), (9, 1), (3, 77)]
    wl = _custom("full_rank", n, edges, w, shapes, 16, 1, sigma=0.3)
    X0 = wl.all_params()
    _check(wl, 1, TOL_1)
    gb = _gb(wl)
    gb.round()
    Wm = np.zeros((n, n))
    for a, b in edges:
        Wm[a, b] = Wm[b, a] = np.float64(np.float32(w))
    Wm += np.diag(1 - Wm.sum(1))
    for l in range(len(shapes)):
        dense = np.einsum("ij,jpq->ipq", Wm, np.stack([X0[i][l].astype(np.float64) for i in range(n)]))
        for i in range(n):
            assert rel_err(gb.get_layer(i, l), dense[i]) <= TOL_1, (l, i)
    gb.close()


@pytest.mark.parametrize("rank,steps", [(8, 2), (6, 1), (12, 1)])
def test_torus_beyond_sixteen_stacked_columns(rank, steps):
    """The appendix 'Changing rank vs changing # power iterations' runs rank 8; on a degree-4
    graph that is 32 stacked columns per worker: two groups of two edges (rank 6: 24 columns in
    groups of 12; rank 12: four groups of one edge)."""
    shapes = [(120, 262), (33, 12), (40, 1), (70, 650), (64, 40)]
    wl = _custom(f"torus3x3_r{rank}", 9, W.torus_edges(3, 3), 1 / 5, shapes, rank, steps)
    _check(wl, 1, TOL_1)
    _check(wl, 3, TOL_10, fused=True, two_calls=True)
    _check_sgd(_custom(f"torus3x3_r{rank}_sgd", 9, W.torus_edges(3, 3), 1 / 5, shapes, rank, 1), [0.1, 0.05], TOL_10)
    if rank <= 8:
        _check_iterate(_custom(f"torus3x3_r{rank}_iter", 9, W.torus_edges(3, 3), 1 / 5, shapes, rank, 1),
                       [1, 2, 1], TOL_10, eta=0.05)


# ------------------------------------------------------------------ peaky spectra
PEAKY_SHAPES = [(130, 262), (75, 40), (300, 27), (33, 1)]
PEAKY_TOPO = {"ring": (5, W.ring_edges(5), 0.05), "torus": (9, W.torus_edges(3, 3), 0.03),
              "path": (3, [[0, 1], [1, 2]], 0.05), "pair": (2, [[0, 1]], 0.05)}


def _planted(topo, rank, gap, steps):
    """sigma_1 = 200, sigma_2 = sigma_1 / gap, then a gentle geometric tail so that all `rank`
    columns have a direction of their own, above a noise floor of ~4e-5; small mixing weights so
    that ten rounds do not gossip the planted part away."""
    n, edges, w = PEAKY_TOPO[topo]
    tail = {2: 2.0, 4: 2.0, 8: 1.5, 16: 1.25}[rank]
    spectrum = [200.0] + [200.0 / gap / tail ** k for k in range(rank - 1)]
    ew = np.full((len(edges),), w, dtype=np.float32)
    return W.Workload(f"peaky_{topo}_r{rank}_gap{gap:g}_s{steps}", n, np.asarray(edges, dtype=np.int32).reshape(-1, 2),
                      ew, PEAKY_SHAPES, rank, steps, 1e-6, 10, 11, tuple(spectrum))


@pytest.mark.parametrize("topo,rank,gap", [
    ("ring", 2, 10.0), ("ring", 2, 1e3), ("ring", 2, 1e4), ("torus", 2, 1e4),
    ("ring", 4, 10.0), ("ring", 4, 1e3), ("torus", 4, 10.0), ("torus", 4, 1e3),
    ("path", 8, 10.0), ("path", 8, 1e3), ("pair", 16, 10.0), ("pair", 16, 1e3)])
def test_differences_with_a_planted_fast_decaying_spectrum(topo, rank, gap):
    """The paper's premise (Section 3.1, appendix on power spectra) is a difference with a few
    dominant singular values.  On the first round from a random Q every column of P = D Q is
    dominated by the top singular direction (nearly parallel columns), and warm-started columns
    have lengths sigma_k^2 spread over many orders of magnitude: the two places where an
    orthonormalisation through the Gram matrix could part from the oracle's left-to-right
    Gram-Schmidt.  Ranks 2-8 take the Gram route, 16 the column-by-column kernel.
      (a) the cold first round, everything at the one-round tolerance;
      (b) six warm power steps on frozen parameters, one update, the same;
      (c) ten warm-started rounds.  Parameters, state and flags at the ten-round tolerance.
          Phat of the small columns is NOT a well-conditioned function of the inputs there: the
          parameters are rounded to float after every round (ulp ~2e-7) while sigma_k of the
          difference is 1e-2 and less, so two runs whose roundings part anywhere drift apart in
          Phat_k by about ulp * sqrt(p) / sigma_k (1e-4 ... 1e-3; the oracle's own steps redone
          in another summation order show the same drift).  So: column 1 at the tolerance, all
          columns when gap = 10, and the GPU's columns orthonormal to 1e-6 in every case."""
    _check(_planted(topo, rank, gap, 1), 1, TOL_1)
    _check(_planted(topo, rank, gap, 6), 1, TOL_1)
    wl = _planted(topo, rank, gap, 1)
    layers = list(range(len(wl.shapes)))
    print(f"case {wl.name} ten rounds", flush=True)
    X, Q = wl.all_params(), wl.all_q()
    gb = _gb(wl, layers, (X, Q))
    gb.run(10)
    info = oracle_rounds(wl, X, Q, 10, layers)
    worst = compare_state(gb, X, Q, layers, TOL_10, what=wl.name, flags=info.degenerate,
                          phat=info.phat if gap == 10.0 else None)
    drift = 0.0
    for l in layers:
        for e in range(gb.n_edges):
            ph = gb.get_phat(e, l).astype(np.float64)
            keep = info.degenerate[l][e] == 0
            assert rel_err(ph[0], info.phat[e][l][0]) <= TOL_10
            gram = ph[keep] @ ph[keep].T
            assert np.abs(gram - np.eye(int(keep.sum()))).max() <= 1e-6
            drift = max(drift, rel_err(ph, info.phat[e][l]))
    print("   worst rel err", worst, "Phat, all columns:", drift, flush=True)
    gb.close()


@pytest.mark.parametrize("factor,dropped", [(0.5, 1), (2.0, 0)])
def test_second_column_just_below_and_just_above_the_drop_threshold(factor, dropped):
    """A column is dropped when its Gram-Schmidt residual has squared norm below 1e-10 of its
    squared norm before projection.  D = s1 u1 v1^T + s2 u2 v2^T with Q = [v1 + v2, v1] makes
    that ratio (s2 / s1)^2, set to half and to twice the threshold: the GPU (which reads the
    residual off the factored Gram matrix) and the oracle (which measures it) must decide alike,
    and agree on every stored value."""
    from paper_2008_01425_amd.device import GossipBuffers
    from oracle import pg_oracle as O
    rng = np.random.default_rng(8)
    p, q = 96, 72
    u, _ = np.linalg.qr(rng.standard_normal((p, 2)))
    v, _ = np.linalg.qr(rng.standard_normal((q, 2)))
    s1 = 8.0
    s2 = s1 * np.sqrt(1e-10 * factor)
    D = s1 * np.outer(u[:, 0], v[:, 0]) + s2 * np.outer(u[:, 1], v[:, 1])
    Xb = np.zeros((p, q), np.float32)
    Xa = D.astype(np.float32)
    Q0 = np.stack([v[:, 0] + v[:, 1], v[:, 0]]).astype(np.float32)
    prob = O.Problem(2, np.array([[0, 1]]), np.array([0.5]), [(p, q)], 2, 1)
    X, Q = [[Xa.copy()], [Xb.copy()]], [[Q0.copy()]]
    info = O.gossip_round(prob, X, Q, want_phat=True)
    assert info.degenerate[0].tolist() == [[0, dropped]]       # the construction puts the oracle where intended
    gb = GossipBuffers(2, [[0, 1]], [0.5], [(p, q)], 2, 1)
    gb.set_layer(0, 0, Xa); gb.set_layer(1, 0, Xb); gb.set_q(0, 0, Q0)
    gb.round()
    assert gb.get_flags(0, 0).tolist() == [0, dropped]
    compare_state(gb, X, Q, [0], TOL_1, what=f"threshold x{factor}", phat=info.phat, flags=info.degenerate)
    gb.close()


# ------------------------------------------------------------------ fallbacks and bad values
def test_sixteen_stacked_columns_on_the_vector_kernels():
    """The kernels that serve 16 stacked columns when the matrix-core passes are switched off
    (and for layers too large for their 32-bit addressing): wide row kernel, split update and
    sweep in fused runs, vector column kernel."""
    old = {k: os.environ.get(k) for k in ("PG_MFMA_ROWS", "PG_MFMA_COLS")}
    os.environ["PG_MFMA_ROWS"] = "0"
    os.environ["PG_MFMA_COLS"] = "0"
    try:
        edges = [[0, 1], [0, 2], [3, 0], [0, 4], [2, 1]]
        shapes = [(50, 131), (17, 70), (100, 64), (9, 3), (33, 200), (16, 65), (1, 40)]
        wl = _custom("star16_vector", 5, edges, [0.2, 0.2, 0.2, 0.2, 0.15], shapes, 4, 2)
        _check(wl, 1, TOL_1)
        _check(wl, 3, TOL_10, fused=True)
        wl = _custom("torus3x3_vector", 9, W.torus_edges(3, 3), 1 / 5, [(200, 650), (33, 12), (40, 1)], 4, 2)
        _check(wl, 1, TOL_1)
        _check(wl, 4, TOL_10, fused=True)
        wl = _custom("torus3x3_vector_sgd", 9, W.torus_edges(3, 3), 1 / 5, [(200, 650), (33, 12), (40, 1)], 4, 1)
        _check_sgd(wl, [0.1, 0.1], TOL_10)
    finally:
        for k, v in old.items():
            if v is None:
                os.environ.pop(k, None)
            else:
                os.environ[k] = v


@pytest.mark.parametrize("mode", ["0", "2"])
def test_vector_layers_with_and_without_kernels_of_their_own(mode):
    """Vector layers (q = 1) run either as tiles of the matrix kernels or, where a parameter set
    has many of them, in launches of their own; both ways against the oracle, on a ring (two
    stacked columns), a torus (four) and with the gradient term, with vectors long enough for
    several steps per lane and a ragged end."""
    old = os.environ.get("PG_VEC_KERNELS")
    os.environ["PG_VEC_KERNELS"] = mode
    try:
        shapes = [(700, 1), (64, 48), (2049, 1), (37, 1), (20001, 1), (256, 1), (16, 130)]
        wl = _custom("ring5_vectors", 5, W.ring_edges(5), 1 / 3, shapes, 2, 1)
        _check(wl, 1, TOL_1)
        _check(wl, 10, TOL_10, fused=True)
        wl = _custom("torus3x3_vectors", 9, W.torus_edges(3, 3), 1 / 5, shapes, 1, 2)
        _check(wl, 1, TOL_1)
        _check(wl, 4, TOL_10, fused=True)
        _check_sgd(wl, [0.1, 0.05], TOL_10)
        wl = _custom("torus3x3_vectors_iter", 9, W.torus_edges(3, 3), 1 / 5, shapes, 1, 1)
        _check_iterate(wl, [1, 1, 2], TOL_10, eta=0.05)
    finally:
        if old is None:
            os.environ.pop("PG_VEC_KERNELS", None)
        else:
            os.environ["PG_VEC_KERNELS"] = old


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_non_finite_values_stay_in_their_layer(bad):
    """A NaN or an infinity in one worker's copy of one layer: the calls still succeed, the value
    is still there afterwards, and every other layer comes out bit for bit as without it
    (layers never mix: Section 2)."""
    wl = _custom("poison", 6, W.ring_edges(6), 1 / 3, [(40, 36), (64, 130), (20, 1), (31, 27)], 2, 2)
    clean, dirty = _gb(wl), _gb(wl)
    x = dirty.get_layer(2, 1)
    x[7, 11] = bad
    dirty.set_layer(2, 1, x)
    for gb in (clean, dirty):
        gb.round()
        gb.run(3)
    assert not np.isfinite(dirty.get_layer(2, 1)).all()
    for l in (0, 2, 3):
        for i in range(6):
            assert np.array_equal(clean.get_layer(i, l), dirty.get_layer(i, l))
        for e in range(6):
            assert np.array_equal(clean.get_q(e, l), dirty.get_q(e, l))
    clean.close(); dirty.close()


def test_single_iterations_on_degenerate_differences():
    """pg_iterate where a stored vector cannot be normalised: identical workers (the odd iteration
    stores a zero vector, the even one drops it and leaves the R^q buffer alone) and a rank-one
    difference at rank 2 (the even iteration drops the second column).  Flags, both buffers and
    the parameters against the oracle."""
    same = _custom("iter_same", 4, W.ring_edges(4), 1 / 3, [(40, 24), (12, 1), (9, 70)], 2, 1, sigma=0.0)
    _check_iterate(same, [1, 1, 1], TOL_10)
    _check_iterate(same, [2, 2], TOL_10)
    from paper_2008_01425_amd.device import GossipBuffers
    from oracle import pg_oracle as O
    rng = np.random.default_rng(5)
    p, q = 48, 40
    base = np.round(rng.standard_normal((p, q)) * 64).astype(np.float32) / 64
    u = rng.integers(-3, 4, p).astype(np.float32)
    v = rng.integers(-3, 4, q).astype(np.float32)
    Xa, Xb = (base + np.outer(u, v) / 64).astype(np.float32), base.copy()   # exactly rank one in float
    V0 = rng.standard_normal((2, q)).astype(np.float32)
    gb = GossipBuffers(2, [[0, 1]], [0.5], [(p, q)], 2, 1)
    gb.alloc_pstate()
    gb.set_layer(0, 0, Xa); gb.set_layer(1, 0, Xb); gb.set_q(0, 0, V0)
    gb.iterate(0, 2)
    prob = O.Problem(2, np.array([[0, 1]]), np.array([0.5]), [(p, q)], 2, 1)
    X, Vq, Vp = [[Xa.copy()], [Xb.copy()]], [[V0.copy()]], [[np.zeros((2, p), np.float32)]]
    drop = O.alg2_round(prob, X, Vq, Vp, 0, 2)
    assert drop[0].tolist() == [[0, 1]]
    assert gb.get_flags(0, 0).tolist() == [0, 1]
    assert np.array_equal(gb.get_q(0, 0)[1], V0[1])
    compare_state(gb, X, Vq, [0], TOL_1, what="iterate rank one")
    assert rel_err(gb.get_p(0, 0), Vp[0][0]) <= TOL_1
    gb.close()


# ------------------------------------------------------------------ extreme aspect ratios
@pytest.mark.parametrize("topo,rank", [("ring", 2), ("torus", 4)])
def test_very_wide_very_tall_and_one_by_one_layers(topo, rank):
    """Rows of 100003 floats (many column segments, odd length), 300001 rows of 3 (many row tiles
    and orthonormalisation chunks), a 1 x 1 layer, two rows of 65537: on the narrow kernels (ring)
    and on the 16-column ones (torus)."""
    n, edges, w = (3, W.ring_edges(3), 1 / 3) if topo == "ring" else (9, W.torus_edges(3, 3), 1 / 5)
    shapes = [(5, 100003), (300001, 3), (1, 1), (2, 65537), (70001, 1)]
    wl = _custom(f"aspect_{topo}", n, edges, w, shapes, rank, 1)
    _check(wl, 1, TOL_1)
    _check(wl, 2, TOL_10, fused=True)


# ------------------------------------------------------------------ maximum sizes
def test_one_layer_of_two_to_the_thirty_elements():
    """A 32768 x 32768 layer: 4 GiB per worker, byte offsets past 2^32 inside one matrix, 64-bit row
    arithmetic in every pass, partial sums of 32768 rows and columns.  Two workers, one edge,
    rank 1, one round and a fused second one; inputs are a random 2048 x 32768 block repeated
    (drawing 3 x 2^30 normals would take longer than the rest of the test)."""
    from paper_2008_01425_amd.device import GossipBuffers
    from oracle import pg_oracle as O
    p = q = 32768
    rng = np.random.default_rng(77)
    t0 = time.time()
    reps = p // 2048

    def big(scale, shift):
        blk = rng.standard_normal((2048, q), dtype=np.float32) * np.float32(scale)
        a = np.tile(blk, (reps, 1))
        # make the repeats differ: a smooth factor per row block
        a *= (1.0 + shift * np.repeat(np.arange(reps, dtype=np.float32), 2048))[:, None]
        return a
    base = big(1.0, 0.01)
    Xa = base + big(0.01, 0.03)
    Xb = base + big(0.01, 0.05)
    del base
    Q0 = rng.standard_normal((1, q)).astype(np.float32)
    print(f"case 2^30 elements: inputs {time.time() - t0:.0f} s", flush=True)
    gb = GossipBuffers(2, [[0, 1]], [0.4], [(p, q)], 1, 1)
    assert gb.N == p * q
    gb.set_layer(0, 0, Xa); gb.set_layer(1, 0, Xb); gb.set_q(0, 0, Q0)
    gb.run(2)
    print(f"   GPU rounds queued {time.time() - t0:.0f} s", flush=True)
    prob = O.Problem(2, np.array([[0, 1]]), np.array([np.float64(np.float32(0.4))]), [(p, q)], 1, 1)
    X, Q = [[Xa], [Xb]], [[Q0]]
    for t in range(2):
        info = O.gossip_round(prob, X, Q, want_phat=True)
        print(f"   oracle round {t + 1} {time.time() - t0:.0f} s", flush=True)
    for i in range(2):
        got = gb.get_layer(i, 0)
        # strided check of the whole matrix plus its last rows and columns, element by element
        for sl in (np.s_[::7, ::5], np.s_[-64:, :], np.s_[:, -64:]):
            assert rel_err(got[sl], X[i][0][sl]) <= TOL_1, (i, sl)
        del got
    assert rel_err(gb.get_q(0, 0), Q[0][0]) <= TOL_1
    assert rel_err(gb.get_phat(0, 0), info.phat[0][0]) <= TOL_1
    assert np.array_equal(gb.get_flags(0, 0), info.degenerate[0][0])
    print(f"   done {time.time() - t0:.0f} s", flush=True)
    gb.close()


# ------------------------------------------------------------------ full-size configurations
# Every named configuration, every layer, one and ten rounds, through pg_round and through pg_run
# (tiny and resnet20 above; the oracle's ten rounds take seconds for the VGG-16 shapes, about
# three minutes for the LSTM shapes, whose 33278 x 650 embedding is one serial oracle call).
def test_vgg16_rank1_full_size_every_layer_one_and_ten_rounds():
    _check_named("vgg16_r1")


def test_vgg16_rank2_full_size_every_layer_one_and_ten_rounds():
    _check_named("vgg16_r2")


def test_lstm_full_size_every_layer_one_and_ten_rounds():
    _check_named("lstm")


def test_resnet50_full_size_every_layer_one_and_ten_rounds():
    _check_named("resnet50")


def test_consensus_experiment_on_unstructured_data():
    """Section 5, Figure 1 (left), 100 x 100 Gaussian data on the 8-ring with W_ij = 0.436.
    (a) every variant contracts towards the mean round after round; (b) the library's curves for
    the warm-started and the random-projection variant are the oracle's, replayed from the same
    seeded matrices and projections; (c) with fresh rank-1 projections (delta = 1 / p,
    Section 4.1) the error shrinks per round at least as fast as Theorem 1's 1 - rho * delta."""
    from paper_2008_01425_amd import consensus_experiment as C
    from oracle import pg_oracle as O
    n, p, q, w, rounds = 8, 100, 100, 0.436, 60
    res = C.run(rounds=rounds, every=1)
    for name, curve in res.items():
        errs = [e for _, _, e in curve]
        assert all(b < a for a, b in zip(errs, errs[1:])), name
        assert errs[-1] < 0.9 * errs[0]
    # (b) the oracle on the same inputs, first ten rounds
    def cerr(X):
        x = np.stack([a[0].astype(np.float64) for a in X])
        return float(((x - x.mean(0)) ** 2).sum() / n)
    prob = O.Problem(n, W.ring_edges(n), np.full((n,), np.float64(np.float32(w))), [(p, q)], 1, 1)
    for name in ("power_iteration", "random_projection"):
        X = [[a] for a in C.initial_matrices(n, p, q, 0)]
        states = C.projection_stream(n, 1, q, 0)
        Q = [[a] for a in next(states)]
        for t in range(10):
            assert abs(res[name][t][2] - cerr(X)) <= TOL_10 * cerr(X), (name, t)
            if name == "random_projection":
                Q = [[a] for a in next(states)]
            O.gossip_round(prob, X, Q)
    # (c) Theorem 1
    Wm = np.zeros((n, n))
    for a, b in W.ring_edges(n):
        Wm[a, b] = Wm[b, a] = w
    Wm += np.diag(1 - Wm.sum(1))
    lam = np.sort(np.abs(np.linalg.eigvalsh(Wm)))[::-1]
    rho, delta = 1 - lam[1] ** 2, 1.0 / p
    errs = [e for _, _, e in res["random_projection"]]
    per_round = (errs[-1] / errs[0]) ** (1.0 / rounds)
    assert per_round <= 1 - rho * delta + 0.002
    assert per_round >= 1 - 6 * rho * delta          # and a rank-1 step cannot contract like full gossip
