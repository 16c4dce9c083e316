"""The work this library is measured on: gossip rounds as a training or consensus program calls them.

A case names the layers of the model (its list of p x q matrices), the graph the workers sit on, the
rank and the power steps, and the entry point the program calls.  Parameters are a common point plus
each worker's own deviation from it, the situation gossip meets while workers train; projection
vectors start as N(0, 1), gradients are small against the parameters."""
import math

import numpy as np
import torch

from paper_2008_01425_amd import binding as B
from paper_2008_01425_amd import workloads as W
from paper_2008_01425_amd.device import GossipBuffers

ETA = 0.05         # learning rate of the calls that take a gradient
GRAD_SCALE = 0.02  # standard deviation of the gradients


def listed():
    """Smallest calls first."""
    def case(name, call, layers, graph, rank, steps, **more):
        return dict(name=name, call=call, layers=layers, graph=graph, rank=rank, steps=steps, sigma=0.01, **more)
    return [
        # one round over three small layers: nothing but latency and launches
        case("tiny_round", "round", "64x32,32x16,16x1", "ring:4", 1, 1),
        # the averaging experiment: one 100 x 100 matrix per worker, many rounds with nothing in between
        case("consensus_run", "run", "100x100", "ring:8", 1, 1, rounds=10),
        # the training step of a small image model, 59 layers, most of them short vectors
        case("resnet20_sgd", "sgd", "resnet20", "ring:8", 1, 1),
        # the same model between evaluations: several gossip rounds per call
        case("resnet20_run", "run", "resnet20", "ring:8", 1, 1, rounds=10),
        # the headline benchmark: consecutive rounds over a large convolutional model
        case("vgg16_run", "run", "vgg16", "ring:16", 1, 1, rounds=10),
        # the same model's training step
        case("vgg16_sgd", "sgd", "vgg16", "ring:16", 1, 1),
        # one gossip round at the next rank
        case("vgg16_r2_round", "round", "vgg16", "ring:16", 2, 1),
        # the cheapest setting in communication: a single matrix-vector iteration per training step
        case("vgg16_iterate", "iterate", "vgg16", "ring:16", 1, 1),
        # a language model on a torus, four columns and two power steps: consecutive rounds ...
        case("lstm_run", "run", "lstm", "torus:4x4", 4, 2, rounds=2),
        # ... and the training step
        case("lstm_sgd", "sgd", "lstm", "torus:4x4", 4, 2),
        # the largest set: 64 workers on a torus, 161 layers
        case("resnet50_round", "round", "resnet50", "torus:8x8", 2, 2),
        # layers of odd lengths on a graph with hubs and leaves
        case("ragged_sgd", "sgd", "510x1023,77x4099,1301x333,2047x255,33x1,129x2,5x70001,40001x7", "tree:11", 3, 1),
    ]


def draw(rng):
    """One more case: any entry point, graph and rank, from one small matrix to hundreds of millions
    of parameters."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    rank = rng.choice([1, 1, 1, 2, 2, 3, 4, 8])
    kind = rng.choice(["ring", "ring", "torus", "tree"])
    if kind == "torus":
        rows, cols = rng.randint(3, 5), rng.randint(3, 5)
        n, graph = rows * cols, "torus:%dx%d" % (rows, cols)
    else:
        n = rng.randint(3, 24)
        graph = "%s:%d" % (kind, n)
    budget = size(2e4, 4e8) / n        # parameters of one worker
    layers, total = [], 0
    for k in range(rng.choice([1, 3, 8, 20, 60])):
        p, q = size(32, 4096), size(32, 8192)
        if k > 0 and rng.random() < 0.3:
            q = rng.choice([1, 1, 3, 7])   # a bias, a normalisation scale, a narrow matrix
        elif rng.random() < 0.5:
            q = 9 * max(4, q // 9)         # a 3 x 3 convolution
        if p * q > budget - total:         # as much of it as is left
            if k > 0:
                break
            f = math.sqrt((budget - total) / (p * q))
            p, q = max(32, int(p * f)), max(32, int(q * f))
        layers.append("%dx%d" % (p, q))
        total += p * q
    call = rng.choice(["round", "sgd", "sgd", "run", "iterate"])
    case = dict(call=call, layers=",".join(layers), graph=graph, rank=rank, steps=rng.choice([1, 1, 2]),
                sigma=rng.choice([0.01, 0.1]))
    if call == "run":
        case["rounds"] = rng.choice([2, 5, 10])
    return case


def shapes_of(case):
    named = {"resnet20": W.resnet20_shapes, "vgg16": W.vgg16_shapes, "lstm": W.lstm_shapes, "resnet50": W.resnet50_shapes}
    if case["layers"] in named:
        return named[case["layers"]]()
    return [tuple(int(v) for v in s.split("x")) for s in case["layers"].split(",")]


def graph_of(case):
    """(workers, edges, mixing weights): 1 / (1 + largest degree of the two ends), as on a regular graph."""
    kind, arg = case["graph"].split(":")
    if kind == "ring":
        n = int(arg)
        edges = W.ring_edges(n)
    elif kind == "torus":
        r, c = (int(v) for v in arg.split("x"))
        n, edges = r * c, W.torus_edges(r, c)
    else:                              # a tree of triples: worker v hangs on (v - 1) // 3
        n = int(arg)
        edges = np.array([[(v - 1) // 3, v] for v in range(1, n)], dtype=np.int32)
    deg = np.bincount(edges.reshape(-1), minlength=n)
    return n, edges, (1.0 / (1 + np.maximum(deg[edges[:, 0]], deg[edges[:, 1]]))).astype(np.float32)


class State:
    """What a program holds: the context, every worker's parameters (one allocation), the projection
    state, the workspace and, where the call takes them, gradients and the other half of the vectors."""

    def __init__(self, case, seed):
        self.call, self.rounds, self.k = case["call"], case.get("rounds", 1), 0
        n, edges, w = graph_of(case)
        self.gb = gb = GossipBuffers(n, edges, w, shapes_of(case), case["rank"], case["steps"])
        gen = torch.Generator(device=gb.device).manual_seed(seed)

        def per_worker():
            flat = torch.empty(n, gb.N, dtype=torch.float32, device=gb.device)
            return flat, list(flat), [t.data_ptr() for t in flat]

        self.x, gb.x, gb.ptrs = per_worker()
        base = torch.empty(gb.N, dtype=torch.float32, device=gb.device).normal_(generator=gen)
        for x in gb.x:
            x.normal_(generator=gen).mul_(case["sigma"]).add_(base)
        gb.q.normal_(generator=gen)
        self.out = [self.x, gb.q]
        if self.call in ("sgd", "iterate"):
            self.g, gb.g, gb.gptrs = per_worker()
            for g in gb.g:
                g.normal_(generator=gen).mul_(GRAD_SCALE)
        if self.call == "iterate":
            gb.alloc_pstate()
            self.out.append(gb.pstate)

    def __del__(self):
        if hasattr(self, "gb"):
            self.gb.close()


def prepare(case, seed):
    return State(case, seed)


def run(state):
    gb = state.gb
    if state.call == "round":
        gb.round()
    elif state.call == "run":
        gb.run(state.rounds)
    elif state.call == "sgd":
        gb.round_sgd(ETA)
    else:
        gb.iterate(state.k, 1, ETA)
        state.k += 1
    return state.out


def exact(case, seed):
    """The same pass with every product, vector and parameter in float64, one layer at a time, all
    edges side by side; buffers laid out as the call leaves them."""
    state = prepare(case, seed)
    gb, call = state.gb, state.call
    _, edges, w = graph_of(case)
    a, b = (torch.as_tensor(edges[:, k].copy(), dtype=torch.int64, device=gb.device) for k in (0, 1))
    w = torch.as_tensor(w, device=gb.device).double().view(-1, 1, 1)
    X, q = state.x.double(), gb.q.double()
    pst = gb.pstate.double() if call == "iterate" else None
    eta = float(np.float32(ETA))

    def unit(V):
        """Gram-Schmidt, left to right; a column without a direction of its own becomes zero."""
        keep, out = [], []
        for k in range(V.shape[2]):
            v = V[:, :, k]
            before = v.square().sum(1)
            for u in out:
                v = v - (u * v).sum(1, keepdim=True) * u
            after = v.square().sum(1)
            ok = after >= torch.clamp(1e-10 * before, min=float(np.finfo(np.float32).tiny))
            out.append(torch.where(ok[:, None], v / after.sqrt()[:, None], torch.zeros_like(v)))
            keep.append(ok)
        return torch.stack(out, 2), torch.stack(keep, 1)[:, None, :]

    for l, ((p, n), r) in enumerate(zip(gb.shapes, gb.ranks)):
        off, ld = B.pg_layer_offset(gb.ctx, l), B.pg_layer_stride(gb.ctx, l)
        at = [B.pg_q_offset(gb.ctx, e, l) for e in range(gb.n_edges)]
        Xl = X[:, off:off + p * ld].view(-1, p, ld)[:, :, :n]
        Q = torch.stack([q[o:o + r * n].view(r, n).T for o in at])      # edge, column of X, column of Q
        for _ in range(state.rounds):
            D = Xl[a] - Xl[b]
            if call == "iterate":          # the first iteration of a new state is an odd one
                right, ok = unit(Q)
                left = D @ right
                pstate = torch.where(ok, left, torch.zeros_like(left))
            else:
                for _ in range(case["steps"]):
                    left, ok = unit(D @ Q)
                    Q = torch.where(ok, D.transpose(1, 2) @ left, Q)
                right = Q
            U = w * (left @ right.transpose(1, 2))
            Xl.index_add_(0, a, U, alpha=-1.0)
            Xl.index_add_(0, b, U)
            del D, U
        if call in ("sgd", "iterate"):
            Xl -= eta * state.g[:, off:off + p * ld].view(-1, p, ld)[:, :, :n].double()
        for e, o in enumerate(at):
            q[o:o + r * n] = Q[e].T.reshape(-1)
            if pst is not None:
                o = B.pg_p_offset(gb.ctx, e, l)
                pst[o:o + r * p] = pstate[e].T.reshape(-1)
    return [X, q] + ([pst] if pst is not None else [])


def work(case):
    """Bytes: every worker's parameters read and written once, gradients and projection vectors read
    once, the new vectors written once, however many rounds the call makes.  Operations: per edge
    and product one difference and a multiply-add per column, per edge end a multiply-add per column
    of the update."""
    n, edges, _ = graph_of(case)
    shapes, r, E = shapes_of(case), case["rank"], len(edges)
    params = float(sum(p * q for p, q in shapes))
    vectors = float(sum(min(r, p, q) * q for p, q in shapes))
    nbytes = 4.0 * (2 * n * params + 2 * E * vectors)
    if case["call"] in ("sgd", "iterate"):
        nbytes += 4.0 * n * params
    products = 1 if case["call"] == "iterate" else 2 * case["steps"]
    flops = E * sum(p * q * (1.0 + 2.0 * min(r, p, q) * (products + 2)) for p, q in shapes) * case.get("rounds", 1)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Four times the difference between one or two passes in float storage and the same steps in
    float64 throughout, over the listed cases and forty drawn ones: one round, 6.7e-6 in norm and
    6.6e-5 at most (all of it in the projection state: each round rounds X, and the next product
    sees that against the much smaller difference of two workers); ten rounds per pass, 2.5e-4 and
    4.1e-3."""
    rounds = case.get("rounds", 1)
    return {"rel": 1e-5 * (2 + rounds ** 2), "max": 1.6e-4 * (1 + rounds ** 2)}
