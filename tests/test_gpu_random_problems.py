"""Seeded random problems -- topology, layer shapes, rank, power steps, call pattern -- on the HIP
path against the CPU oracle: the corners the hand-picked cases may miss (mixed degrees with and
without column groups, isolated workers, rows of every alignment, one-row and one-column layers,
ranks above a dimension)."""
import numpy as np
import pytest

from paper_2008_01425_amd import workloads as W
from parity_util import PATHS, TOL_1, TOL_10, compare_state, env_settings, launched, oracle_rounds

pytestmark = pytest.mark.gpu


def _random_problem(seed):
    rng = np.random.default_rng([2008, 1425, seed])
    n = int(rng.integers(2, 10))
    # a random spanning tree plus a few chords (or, sometimes, one worker left without edges)
    lone = n > 3 and rng.random() < 0.2
    m = n - 1 if lone else n
    order = rng.permutation(m)
    edges = set()
    for k in range(1, m):
        a, b = int(order[k]), int(order[int(rng.integers(0, k))])
        edges.add((a, b) if rng.random() < 0.5 else (b, a))
    for _ in range(int(rng.integers(0, m + 1))):
        a, b = (int(v) for v in rng.integers(0, m, 2))
        if a != b and (a, b) not in edges and (b, a) not in edges:
            edges.add((a, b))
    edges = sorted(edges)
    deg = np.bincount(np.asarray(edges).reshape(-1), minlength=n)
    # weights: positive, every worker's sum at most 1
    w = np.array([rng.uniform(0.3, 1.0) / max(deg[a], deg[b]) for a, b in edges], np.float32)
    # well-conditioned shapes: rank well below both dimensions for most layers, plus odd ones
    pool = [(int(rng.integers(40, 300)), int(rng.integers(40, 700))) for _ in range(3)]
    pool += [(int(rng.integers(1, 40)), int(rng.integers(1, 40))) for _ in range(2)]
    pool += [(int(rng.integers(1, 2000)), 1), (1, int(rng.integers(1, 300)))]
    shapes = [pool[i] for i in rng.permutation(len(pool))[:int(rng.integers(2, 6))]]
    rank = int(rng.choice([1, 1, 2, 2, 3, 4, 5, 8]))
    steps = int(rng.choice([1, 1, 2, 3]))
    return W.Workload(f"random{seed}", n, np.asarray(edges, np.int32).reshape(-1, 2), w, shapes, rank, steps,
                      float(rng.choice([0.02, 0.1, 0.5])), 10, 1000 + seed)


def _of_path(path, seed):
    """The problem of this seed; for edge kernels of its small layers, at most rank 4."""
    wl = _random_problem(seed)
    if path == "edge kernels":
        small = [s for s in wl.shapes if s[0] * s[1] <= 512 * 4 and s[0] <= 512] or [(40, 37)]
        wl = W.Workload(wl.name, wl.n_workers, wl.edges, wl.edge_w, small, min(wl.rank, 4), wl.power_steps, wl.sigma, 10, 1000 + seed)
    return wl


@pytest.mark.parametrize("seed", range(24))
def test_random_problem_one_round_and_a_short_fused_run(seed):
    # even seeds with the row blocking of large parameter sets, odd seeds with that of small ones
    # (by size all of these problems would get the latter)
    _round_and_run(_random_problem(seed), dict(PG_LIGHT=seed % 2))


@pytest.mark.parametrize("path", ["by rule", "edge kernels", "edge sweeps"])
@pytest.mark.parametrize("seed", range(24))
def test_random_problem_one_round_and_a_short_run_on_other_kernels(seed, path):
    wl = _of_path(path, seed)
    kinds = _round_and_run(wl, PATHS.get(path, {}))
    if path == "edge kernels":
        assert "edge" in kinds, kinds
    if path == "edge sweeps" and wl.rank <= 4:
        assert "edge_sweep" in kinds, kinds


def _round_and_run(wl, settings):
    from paper_2008_01425_amd.device import GossipBuffers
    layers = list(range(len(wl.shapes)))
    print(f"case {wl.name}: n={wl.n_workers} edges={wl.edges.tolist()} shapes={wl.shapes} rank={wl.rank} "
          f"steps={wl.power_steps} sigma={wl.sigma} {settings}", flush=True)
    X, Q = wl.all_params(), wl.all_q()
    with env_settings(settings):
        a = GossipBuffers.from_workload(wl, fill=False)
        b = GossipBuffers.from_workload(wl, fill=False)
    a.fill_from_arrays(X, Q)
    b.fill_from_arrays(X, Q)
    kinds = launched(a, a.round)
    b.run(2)
    b.round()
    info, snaps = oracle_rounds(wl, X, Q, 3, layers, snap_at=(1,))
    s1 = snaps[1]
    w1 = compare_state(a, s1.X, s1.Q, layers, TOL_1, what=wl.name + " one round", phat=s1.phat, flags=s1.degenerate)
    # three rounds: parameters and flags at the ten-round bar; the state of tiny or nearly
    # full-rank layers is too ill-conditioned on unstructured data to be held to it
    w3 = compare_state(b, X, Q, layers, TOL_10, what=wl.name + " three rounds", flags=info.degenerate, check_q=False)
    print("   worst rel err", w1, w3, flush=True)
    a.close()
    b.close()
    return kinds


@pytest.mark.parametrize("seed", range(100, 112))
def test_random_problem_sgd_step_and_single_iterations(seed):
    _sgd_and_iterations(_random_problem(seed), seed, dict(PG_LIGHT=seed % 2))


@pytest.mark.parametrize("path", ["by rule", "edge kernels", "edge sweeps"])
@pytest.mark.parametrize("seed", range(100, 112))
def test_random_problem_sgd_step_and_single_iterations_on_other_kernels(seed, path):
    _sgd_and_iterations(_of_path(path, seed), seed, PATHS.get(path, {}))


def _sgd_and_iterations(wl, seed, settings):
    """The same random problems through Algorithm 1's step (gradient folded into the update) and
    through Algorithm 2 one iteration at a time (with and without a gradient)."""
    from oracle import pg_oracle as O
    from parity_util import oracle_problem, rel_err
    from paper_2008_01425_amd.device import GossipBuffers
    L, E, n = len(wl.shapes), wl.n_edges, wl.n_workers
    layers = list(range(L))
    print(f"case {wl.name}: n={n} edges={wl.edges.tolist()} shapes={wl.shapes} rank={wl.rank} steps={wl.power_steps}",
          flush=True)
    prob = oracle_problem(wl)
    rng = np.random.default_rng(seed)
    G = [[rng.standard_normal(s).astype(np.float32) for s in wl.shapes] for _ in range(n)]
    eta = 0.05
    # Algorithm 1's step
    X, Q = wl.all_params(), wl.all_q()
    with env_settings(settings):
        gb = GossipBuffers.from_workload(wl, fill=False)
    gb.fill_from_arrays(X, Q)
    gb.alloc_grads()
    for i in range(n):
        for l in layers:
            gb.set_grad_layer(i, l, G[i][l])
    gb.round_sgd(eta)
    O.gossip_round(prob, X, Q, G=G, eta=float(np.float32(eta)))
    w1 = compare_state(gb, X, Q, layers, TOL_1, what=wl.name + " sgd")
    gb.close()
    # Algorithm 2, iterations 1, 2 and 3 in two calls, the second with the gradient
    X, Vq = wl.all_params(), wl.all_q()
    Vp = [[np.zeros((wl.layer_rank(l), wl.shapes[l][0]), np.float32) for l in layers] for _ in range(E)]
    with env_settings(settings):
        gb = GossipBuffers.from_workload(wl, fill=False)
    gb.fill_from_arrays(X, Vq)
    gb.alloc_pstate()
    gb.alloc_grads()
    for i in range(n):
        for l in layers:
            gb.set_grad_layer(i, l, G[i][l])
    gb.iterate(0, 1)
    drop = O.alg2_round(prob, X, Vq, Vp, 0, 1)
    w2 = compare_state(gb, X, Vq, layers, TOL_1, what=wl.name + " iteration 1", flags=drop)
    gb.iterate(1, 2, eta)
    drop = O.alg2_round(prob, X, Vq, Vp, 1, 2, G=G, eta=float(np.float32(eta)))
    w3 = compare_state(gb, X, Vq, layers, TOL_10, what=wl.name + " iterations 2-3", flags=drop, check_q=False)
    for l in layers:
        for e in range(E):
            assert rel_err(gb.get_p(e, l), Vp[e][l]) <= TOL_10, (e, l)
    print("   worst rel err", w1, w2, w3, flush=True)
    gb.close()
