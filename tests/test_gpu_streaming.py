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


def _workload(name, n, edges, rank, steps, sigma=0.05):
    edges = np.asarray(edges, np.int32).reshape(-1, 2)
    deg = np.bincount(edges.reshape(-1), minlength=n)
    w = np.array([1.0 / (1 + max(deg[a], deg[b])) for a, b in edges], np.float32)
    return W.Workload(name, n, edges, w, SHAPES, rank, steps, sigma, 10, 77)


def _buffers(wl, X, Q, stream, lazy):
    from paper_2008_01425_amd.device import GossipBuffers
    with env_setting("PG_STREAM", stream), env_setting("PG_LAZY", lazy), env_setting("PG_LIGHT", 0):
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


@pytest.mark.parametrize("graph", GRAPHS)
@pytest.mark.parametrize("rounds", [2, 3, 4, 7])
@pytest.mark.parametrize("rank", [1, 2])
def test_a_run_that_writes_every_second_round_equals_the_plain_run(graph, rounds, rank):
    n, edges = GRAPHS[graph]
    wl = _workload(f"lazy {graph} {rounds} r{rank}", n, edges, rank, 1)
    X, Q = wl.all_params(), wl.all_q()
    for l in (1, 6):                                   # two neighbours agree: their columns are dropped
        X[1][l] = X[0][l].copy()
    plain, lazy = _buffers(wl, X, Q, 0, 0), _buffers(wl, X, Q, 1, 1)
    for _ in range(2):                                 # the second call starts on what the first left
        plain.run(rounds)
        lazy.run(rounds)
        _same(plain, lazy, wl, wl.name)
    plain.round()
    lazy.round()
    _same(plain, lazy, wl, wl.name + " and one round")
    plain.close()
    lazy.close()


@pytest.mark.parametrize("rank", [1, 2, 3, 4])
def test_streamed_passes_equal_the_cached_ones(rank):
    """1 to 16 stacked columns: every row and column kernel, each call."""
    import torch
    n, edges = 6, [(0, 1), (0, 2), (3, 0), (0, 4), (2, 1), (4, 5)]   # degrees 4, 2, 2, 1, 2, 1
    wl = _workload(f"stream r{rank}", n, edges, rank, 2)
    X, Q = wl.all_params(), wl.all_q()
    a, b = _buffers(wl, X, Q, 0, 0), _buffers(wl, X, Q, 1, 1)
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
