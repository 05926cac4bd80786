"""The work that programs built on this library do, as cases that can be timed.

A p-median program preprocesses distance matrices, evaluates populations, runs
the genetic algorithm (alone, in ragged batches, or with the learned swap
proposal) and, for graph instances, first computes the distances.  The cases
take the shapes of this repository's benchmark and tests (graph instances of
100 and 900 vertices, Euclidean ones of 2000 and 5000 points, ragged batches,
wide instances) and odd sizes between them.

``listed()`` gives the cases, ``draw(rng)`` another one of the same ranges,
``prepare`` what a program holds before the call, ``run`` one pass through the
public entry points, ``work`` the bytes and operations a pass cannot do
without, ``exact`` the same outputs by plain torch in 64 bits.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1610_10061_amd as pm

LEARN = dict(candidates=64, learned_iters=4, explore_permille=50, history=4, lr=2e-3)


def listed():
    return [
        # a program that hands over a small host matrix and wants a solution:
        # graph with 100 vertices, the smallest benchmark configuration
        dict(name="solve_graph100", kind="solve", inst="graph", n=100, m=100, p=5, edges=200,
             population=64, group=64, generations=100),
        # the smallest evaluation call, waited for (a local search that asks
        # for a handful of candidates at a time): latency of one call
        dict(name="eval_graph100", kind="eval", inst="graph", n=100, m=100, p=5, edges=200,
             population=64, wait=True, scan=False),
        # an ordinary population of the graph benchmark, enqueued without a
        # wait (an evolution loop of the program's own)
        dict(name="eval_graph900", kind="eval", inst="graph", n=900, m=900, p=90, edges=16200,
             population=1024, wait=False, scan=False),
        # the largest evaluation: few open facilities, long scans
        dict(name="eval_euclid5000_p10", kind="eval", inst="euclid", n=5000, m=5000, p=10,
             population=4096, wait=False, scan=True),
        # many open facilities, short scans, clients and facilities of
        # different, odd numbers, a population that fills no whole tile
        dict(name="eval_ragged_p333", kind="eval", inst="euclid", n=4801, m=3333, p=333,
             population=4001, wait=True, scan=False),
        # setting an instance up (tables made on the device) and evaluating a
        # first population on it: graph benchmark size, distances below 2^16
        dict(name="setup_graph900", kind="setup", inst="graph", n=900, m=900, p=90, edges=16200,
             population=256),
        # the same at the largest square instance
        dict(name="setup_euclid5000", kind="setup", inst="euclid", n=5000, m=5000, p=100,
             population=256),
        # more facilities than one workgroup's memory sorts, distances past
        # 2^16 (cost matrices in metres)
        dict(name="setup_wide20001", kind="setup", inst="points", n=777, m=20001, p=150,
             population=256),
        # a whole run of the genetic algorithm on an instance in hand: the
        # headline configuration, 100 generations
        dict(name="ga_graph900", kind="ga", inst="graph", n=900, m=900, p=90, edges=16200,
             population=1024, group=256, generations=100),
        # the run with the learned swap proposal, its network trained online
        # (scoring forward, training forward and backward, updated weights)
        dict(name="learned_euclid2000", kind="learned", inst="euclid", n=2000, m=2000, p=200,
             population=1024, group=256, generations=24),
        # ragged instances evolved together
        dict(name="batch_ragged64", kind="batch", count=64, nmin=100, nmax=2000,
             population=256, group=256, generations=20),
        # distances of a graph instance from its edge weights
        dict(name="apsp_graph2000", kind="apsp", n=2000, edges=8000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "eval", "eval", "eval", "setup", "setup", "ga", "learned",
                       "batch", "apsp"])
    if kind == "apsp":
        n = _log_int(rng, 90, 2000)
        return dict(kind=kind, n=n, edges=4 * n)
    if kind == "batch":
        return dict(kind=kind, count=rng.randint(8, 64), nmin=100, nmax=rng.choice([600, 1999]),
                    population=256, group=256, generations=rng.randint(3, 20))
    if kind == "solve":
        n = _log_int(rng, 60, 400)
        return dict(kind=kind, inst="graph", n=n, m=n, p=rng.randint(3, max(4, n // 10)),
                    edges=3 * n, population=64 * rng.randint(1, 4), group=64,
                    generations=rng.randint(20, 100))
    if kind == "learned":
        n = _log_int(rng, 200, 2000)
        return dict(kind=kind, inst="euclid", n=n, m=n, p=max(4, n // rng.randint(8, 16)),
                    population=256 * rng.randint(1, 4), group=256,
                    generations=rng.randint(6, 24))
    if kind == "ga":
        n = _log_int(rng, 100, 900)
        return dict(kind=kind, inst="graph", n=n, m=n, p=max(5, n // rng.randint(8, 20)),
                    edges=4 * n, population=256 * rng.randint(1, 4), group=256,
                    generations=rng.randint(10, 100))
    if kind == "setup":
        if rng.random() < 0.25:
            return dict(kind=kind, inst="points", n=_log_int(rng, 50, 700),
                        m=_log_int(rng, 8193, 20001), p=rng.randint(50, 300), population=256)
        m = _log_int(rng, 100, 5000)
        return dict(kind=kind, inst=rng.choice(["euclid", "points"]), n=_log_int(rng, 100, 5000),
                    m=m, p=rng.randint(5, max(6, m // 8)), population=rng.randint(1, 256))
    m = _log_int(rng, 100, 5000)
    return dict(kind=kind, inst="euclid", n=_log_int(rng, 100, 5000), m=m,
                p=rng.randint(max(3, m // 500), max(4, m // 5)),
                population=_log_int(rng, 64, 4096), wait=rng.random() < 0.5,
                scan=rng.random() < 0.5)


# ------------------------------------------------------------------ inputs
def _euclid(n, m, rng, grid):
    """n x m rounded Euclidean distances of random integer points (clients
    and facilities the same points when n = m), exact, on the GPU."""
    pts = torch.from_numpy(rng.integers(0, grid, size=(n, 2), dtype=np.int64)).cuda()
    sites = pts if n == m else torch.from_numpy(
        rng.integers(0, grid, size=(m, 2), dtype=np.int64)).cuda()
    dx = pts[:, None, 0] - sites[None, :, 0]
    dy = pts[:, None, 1] - sites[None, :, 1]
    s = dx * dx + dy * dy
    r = s.double().sqrt().floor().long()
    r -= (r * r > s).long()
    r += ((r + 1) * (r + 1) <= s).long()
    return (r + ((s - r * r) > r).long()).int().contiguous()


def _weights(n, edges, rng):
    """Arc weights (n x n int32, -1 where there is no edge) of a random
    connected graph: a random spanning tree, then random extra edges."""
    order = rng.permutation(n)
    earlier = order[rng.integers(0, np.arange(1, n))]
    a = np.concatenate([order[1:], rng.integers(0, n, edges - n + 1)])
    b = np.concatenate([earlier, rng.integers(0, n, edges - n + 1)])
    w = rng.integers(1, 101, len(a)).astype(np.int32)
    out = np.full((n, n), -1, np.int32)
    out[a, b] = w
    out[b, a] = w
    np.fill_diagonal(out, 0)
    return torch.from_numpy(out).cuda()


def _shortest_paths(w):
    """Floyd-Warshall in plain torch, 64 bits; -1 where there is no path."""
    far = 1 << 40
    d = torch.where(w < 0, torch.full_like(w, far, dtype=torch.int64), w.long())
    for k in range(d.shape[0]):
        torch.minimum(d, d[:, k:k + 1] + d[k:k + 1, :], out=d)
    return torch.where(d >= far, torch.full_like(d, -1), d)


def _matrix(case, rng):
    if case["inst"] == "graph":
        return _shortest_paths(_weights(case["n"], case["edges"], rng)).int().contiguous()
    grid = 10_000 if case["inst"] == "euclid" else 1_000_000
    return _euclid(case["n"], case["m"], rng, grid)


def _open_bits(case, seed):
    """population x m random 0/1 chromosomes with p ones each (torch bool)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    P, m, p = case["population"], case["m"], case["p"]
    idx = torch.rand((P, m), device="cuda", generator=g).topk(p, dim=1).indices
    bits = torch.zeros((P, m), dtype=torch.bool, device="cuda")
    return bits.scatter_(1, idx, True)


def _pack(bits):
    P, m = bits.shape
    W = (m + 63) // 64
    b = torch.zeros((P, W * 64), dtype=torch.int64, device="cuda")
    b[:, :m] = bits
    shifts = torch.arange(64, dtype=torch.int64, device="cuda")
    return (b.view(P, W, 64) << shifts).sum(2).contiguous().view(torch.uint64)


def _batch_shapes(case):
    """Sizes of a batch's instances: they belong to the case, not the seed."""
    rng = np.random.default_rng([case["count"], case["nmin"], case["nmax"]])
    shapes = []
    for b in range(case["count"]):
        n = int(round(math.exp(rng.uniform(math.log(case["nmin"]), math.log(case["nmax"])))))
        shapes.append(dict(inst="graph" if b % 2 == 0 else "euclid", n=n, m=n,
                           p=int(rng.integers(5, n // 4 + 1)), edges=4 * n))
    return shapes


def prepare(case, seed):
    kind = case["kind"]
    rng = np.random.default_rng([seed, 1610])
    st = {"case": case, "kind": kind, "seed": seed % 1_000_003}
    if kind == "apsp":
        st["w"] = _weights(case["n"], case["edges"], rng)
        st["d"] = torch.empty((case["n"], case["n"]), dtype=torch.int32, device="cuda")
        return st
    if kind == "batch":
        st["shapes"] = _batch_shapes(case)
        st["insts"] = [pm.Instance(_matrix(s, rng), s["p"]) for s in st["shapes"]]
        return st
    d = _matrix(case, rng)
    if kind == "solve":
        st["d"] = d.cpu().numpy()
        return st
    if kind == "setup":
        st["d"] = d
    else:
        st["inst"] = pm.Instance(d, case["p"])
    if kind in ("eval", "setup"):
        st["masks"] = _pack(_open_bits(case, seed))
        P = case["population"]
        st["fitness"] = torch.empty(P, dtype=torch.int64, device="cuda")
        st["scan"] = (torch.empty(P, dtype=torch.int64, device="cuda")
                      if kind == "setup" or case["scan"] else None)
    return st


# --------------------------------------------------------------- one pass
def run(st):
    case, kind = st["case"], st["kind"]
    if kind == "eval":
        st["inst"].eval(st["masks"], st["fitness"], st["scan"],
                        asynchronous=not case["wait"])
        return [st["fitness"]] if st["scan"] is None else [st["fitness"], st["scan"]]
    if kind == "setup":
        inst = pm.Instance(st["d"], case["p"])
        inst.eval(st["masks"], st["fitness"], st["scan"])
        inst.close()
        return [st["fitness"], st["scan"]]
    if kind == "apsp":
        pm.pmp_apsp(st["w"], st["d"])
        return [st["d"]]
    if kind == "solve":
        open_, cost, stats = pm.pmp_solve(st["d"], case["p"], case["population"], case["group"],
                                          case["generations"], st["seed"])
        return [open_, cost, stats]
    if kind == "ga":
        ga = pm.GA(st["inst"], case["population"], case["group"], case["generations"],
                   st["seed"])
        ga.step(case["generations"])
        mask, cost, stats = ga.best()
        population, fitness, group_masks, group_costs = ga.state()
        ga.close()
        return [mask, cost, stats, population, fitness, group_masks, group_costs]
    if kind == "learned":
        model = pm.Model(st["seed"])
        ga = pm.GA(st["inst"], case["population"], case["group"], case["generations"],
                   st["seed"])
        ga.set_model(model, train_every=1, **LEARN)
        ga.step(case["generations"])
        mask, cost, stats = ga.best()
        population, fitness, _, _ = ga.state()
        ga.close()
        weights = model.params()
        model.close()
        return [mask, cost, stats, population, fitness, weights]
    # batch
    gas = [pm.GA(inst, case["population"], case["group"], case["generations"], st["seed"] + b)
           for b, inst in enumerate(st["insts"])]
    batch = pm.Batch(gas)
    batch.autotune()
    batch.step(case["generations"])
    batch.check()
    masks, costs, stats = zip(*[ga.best() for ga in gas])
    batch.close()
    for ga in gas:
        ga.close()
    return [np.concatenate(masks), np.array(costs), np.array([list(s.values()) for s in stats])]


# ------------------------------------------------------------ what it needs
def _ga_pairs(case, n):
    """(client, chromosome) pairs of a run: the population, every crossover
    stage's offspring and one mutation attempt at least per generation."""
    stages = int(math.log2(case["group"]))
    return case["generations"] * case["population"] * n * (2 + stages)


def _table_bytes(n, m, p, population=None):
    """Table entries an evaluation reads: facility index and distance of
    every position up to the farthest scan expected in the population."""
    k = m - p + 1
    if population is not None:
        k = min(k, int(math.ceil(m / p * math.log(max(2.0, population * math.e)))))
    return 6 * n * k


def work(case):
    kind = case["kind"]
    if kind == "apsp":
        n = case["n"]
        return {"bytes": 8 * n * n, "flops": 2 * n ** 3}
    if kind == "batch":
        byts = flops = 0
        for s in _batch_shapes(case):
            byts += _table_bytes(s["n"], s["m"], s["p"])
            flops += _ga_pairs(case, s["n"])
        return {"bytes": byts, "flops": flops}
    n, m, p, P = case["n"], case["m"], case["p"], case["population"]
    mask_bytes = P * ((m + 63) // 64) * 8
    if kind == "eval":
        return {"bytes": _table_bytes(n, m, p, P) + mask_bytes + 8 * P * (1 + case["scan"]),
                "flops": n * P}
    if kind == "setup":
        # d in, the truncated order, gaps and distances out, then the evaluation
        return {"bytes": 4 * n * m + 10 * n * (m - p + 1) + mask_bytes + 16 * P,
                "flops": n * P + n * m * math.ceil(math.log2(m))}
    byts = _table_bytes(n, m, p) + mask_bytes
    flops = _ga_pairs(case, n)
    if kind == "solve":
        byts += 4 * n * m
    if kind == "learned":
        # scoring every candidate, then forward and backward over the ring
        rows = LEARN["learned_iters"] * LEARN["history"]
        flops += case["generations"] * P * 41_200 * (LEARN["candidates"] + 3 * rows)
    return {"bytes": byts, "flops": flops}


# -------------------------------------------------------------- 64-bit values
def exact(case, seed):
    """Evaluations straight from the distances (the least distance to an open
    facility; its place in the order by distance and index), shortest paths by
    Floyd-Warshall.  The runs of the genetic algorithm have no such value:
    they are defined by their random draws."""
    kind = case["kind"]
    rng = np.random.default_rng([seed, 1610])
    if kind == "apsp":
        return [_shortest_paths(_weights(case["n"], case["edges"], rng)).cpu()]
    if kind not in ("eval", "setup"):
        return None
    d = _matrix(case, rng).long()
    n, m = d.shape
    order = (d * m + torch.arange(m, device="cuda")).argsort(dim=1)
    rank = torch.empty_like(order).scatter_(
        1, order, torch.arange(1, m + 1, device="cuda").expand(n, m).contiguous())
    d_t, rank_t = d.t().contiguous(), rank.t().contiguous()
    bits = _open_bits(case, seed)
    fitness = torch.empty(bits.shape[0], dtype=torch.int64, device="cuda")
    scan = torch.empty_like(fitness)
    for c in range(bits.shape[0]):
        where = bits[c].nonzero().squeeze(1)
        fitness[c] = d_t[where].amin(0).sum()
        scan[c] = rank_t[where].amin(0).sum()
    if kind == "setup" or case["scan"]:
        return [fitness.cpu(), scan.cpu()]
    return [fitness.cpu()]
