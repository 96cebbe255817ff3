"""Performance cases: the work a user has this framework do, through its
public entry points.

A case is a dict of plain values.  ``listed()`` gives the named ones,
``draw(rng)`` another of the same ranges.  ``prepare`` makes what a program
holds before the call (a run that has evolved for a while, a pool of admitted
runs, sampled annotations, workspaces and output buffers), ``run`` is one
pass.  Sizes are those of ``paper_2404_10861_amd/workloads.py`` and of the
tests, or generic ones between them.

Paths:
  run    advance one run by ``gens`` generations (ticks) and read its whole
         population back: to the host where it is small, as the whole-
         population sample on the device where it is large
  clade  the clade trial: a fresh run of a tiny torus with founder tags, the
         bounds of the whole population, the tree of one agent per island
  pool   advance a pool of batched runs and read every one's whole population
         as its sample on the device
  serve  a batch of requests through the continuous-batching server, with
         each request's all-pairs bounds on the host
  mrca   all-pairs bounds of a sample (shared or drifted counters)
  tree   the reconstructed tree of a set of annotations, on the host
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

import paper_2404_10861_amd as hs
from paper_2404_10861_amd import serve as srv
from paper_2404_10861_amd import workloads as wl

WARM = 64                  # generations a run has behind it before the first pass
HOST_READ_AGENTS = 4096    # runs up to this size are read back whole to the host
SERVE_SAMPLE = 1024        # agents of a request's all-pairs query (the served workload's figure)
SERVE_POOL_BYTES = 2 << 30


def listed():
    def run(name, w, h, n, sites, kind, gens, **kw):
        case = dict(name=name, path="run", w=w, h=h, n=n, sites=sites, kind=kind, bits=1,
                    interval=1, model="int", tournament=2, migrants=1, activity=0.0, gens=gens)
        case.update(kw)
        return case

    return [
        # the CPU-scale workload: a whole small experiment, the host waiting for it
        run("small_run", 8, 8, 32, 32, "steady", 1000),
        # the clade reconstruction trial: the smallest whole call, all launches and latency
        dict(name="clade_trial", path="clade", w=3, h=3, n=32, sites=64, kind="tilted",
             gens=250),
        # about the median request of the served workload, odd sides
        run("medium_run", 45, 67, 32, 64, "hybrid", 256),
        # the paper-scale run: 16.8 M agents, beyond the last-level cache
        run("paper_scale_run", 512, 1024, 32, 64, "hybrid", 64),
        # one treatment of the pair: one-word surfaces, neutral births, cache-sized
        run("treatment_neutral", 256, 256, 64, 32, "tilted", 128, tournament=0),
        # the on-hardware trial: 18 M agents, binary32 fitness, tournament of five
        run("float_trial", 750, 750, 32, 64, "tilted", 32, model="float", tournament=5),
        # asynchronous ticks on the paper-scale torus: agents keep their own counters
        run("async_ticks", 512, 1024, 32, 64, "hybrid", 40, activity=0.9),
        # the 64 batched runs of mixed sizes, surfaces and treatments, at the tuner's choice
        dict(name="batched_64_runs", path="pool", first=0, runs=64, gens=128, block=256,
             graph=True),
        # requests of the served workload arriving together, bounds delivered to the host
        dict(name="served_requests", path="serve", first=0, requests=8, gens_div=4, chunk=256),
        # the end-of-run query of the treatment pair from annotations alone
        dict(name="mrca_4096", path="mrca", n=4096, sites=32, kind="tilted", bits=1, interval=1,
             activity=0.0, age=2000, bound=False),
        # the same query of an asynchronous run's sample: every pair of another age
        dict(name="mrca_4096_drifted", path="mrca", n=4096, sites=64, kind="hybrid", bits=1,
             interval=1, activity=0.9, age=2000, bound=True),
        # the float trial's 10,000-agent tree
        dict(name="tree_10000", path="tree", n=10000, sites=64, kind="tilted", bits=1,
             interval=1, age=20000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _scheme_draw(rng, horizon_free):
    """(sites, kind, bits, interval): mostly one-bit differentiae on 32 or 64
    sites deposited every generation; sometimes bytes (on a steady surface,
    whose horizon is the counter's) or a coarser interval.  horizon_free
    leaves out the 32-site hybrid surface, which ends after 131,071 items."""
    if rng.random() < 0.15:
        return rng.choice((4, 8)), "steady", 8, rng.choice((1, 3))
    sites = rng.choice((32, 64))
    kinds = ["steady", "tilted", "hybrid"]
    if horizon_free and sites == 32:
        kinds.remove("hybrid")
    return sites, rng.choice(kinds), 1, rng.choice((1, 1, 1, 4))


def draw(rng):
    path = rng.choice(("run",) * 5 + ("clade", "pool", "serve") + ("mrca",) * 2 + ("tree",) * 2)
    if path == "run":
        n = rng.choice((16, 32, 32, 64, rng.randint(1, 64)))
        islands = max(1, _log_int(rng, 64, 1 << 24) // n)
        w = min(islands, max(1, int(math.sqrt(islands) * rng.uniform(0.5, 2.0))))
        h = max(1, islands // w)
        sites, kind, bits, interval = _scheme_draw(rng, True)
        model = rng.choice(("int", "int", "int", "float", "tag"))
        activity = rng.choice((0.0, 0.0, 0.0, round(rng.uniform(0.3, 0.97), 2)))
        most = (1 << 28) if model == "float" or activity else (1 << 29)
        gens = max(8, min(rng.randint(100, 600), most // (w * h * n)))
        return dict(path="run", w=w, h=h, n=n, sites=sites, kind=kind, bits=bits,
                    interval=interval, model=model,
                    tournament={"int": rng.choice((2, 0)), "float": rng.randint(0, 5),
                                "tag": 0}[model],
                    migrants=0 if rng.random() < 0.1 else 1, activity=activity, gens=gens)
    if path == "clade":
        return dict(path="clade", w=rng.randint(2, 6), h=rng.randint(2, 6),
                    n=rng.choice((16, 32, 31)), sites=rng.choice((32, 64)),
                    kind=rng.choice(("steady", "tilted", "hybrid")),
                    gens=rng.choice((25, 50, 100, 250)) + rng.randint(0, 9))
    if path == "pool":
        runs = rng.randint(16, 64)
        return dict(path="pool", first=rng.randint(0, 64 - runs), runs=runs,
                    gens=rng.randint(32, 96), block=rng.choice((64, 128, 256)),
                    graph=rng.random() < 0.5)
    if path == "serve":
        return dict(path="serve", first=rng.randint(0, 2000), requests=rng.randint(2, 8),
                    gens_div=rng.choice((8, 16)), chunk=rng.choice((128, 256)))
    if path == "mrca":
        sites, kind, bits, interval = _scheme_draw(rng, False)
        return dict(path="mrca", n=_log_int(rng, 64, 6000), sites=sites, kind=kind, bits=bits,
                    interval=interval, activity=rng.choice((0.0, round(rng.uniform(0.5, 0.97), 2))),
                    age=_log_int(rng, 100, 4000), bound=rng.random() < 0.5)
    sites, kind, bits, interval = _scheme_draw(rng, False)
    return dict(path="tree", n=_log_int(rng, 64, 16000), sites=sites, kind=kind, bits=bits,
                interval=interval, age=_log_int(rng, 100, 20000))


# ---------------------------------------------------------------------------
def _config(case, seed):
    model = case.get("model", "int")
    extra = {}
    if model == "float":
        extra = dict(del_threshold=wl.P_DELETERIOUS, ben_threshold=wl.P_BENEFICIAL)
    return hs.Config(case["w"], case["h"], case["n"], case["sites"], case["kind"],
                     tournament_size=case.get("tournament", 0), fitness_model=model,
                     migrants_per_island=case.get("migrants", 1), seed=seed + 1,
                     differentia_bits=case.get("bits", 1),
                     ingest_interval=case.get("interval", 1),
                     async_activity=int(case.get("activity", 0.0) * 2**32), **extra)


def _sample_buffers(n, words):
    return (torch.empty(n, dtype=torch.int32, device="cuda"),
            torch.empty(n, dtype=torch.int32, device="cuda"),
            torch.empty((n, words), dtype=torch.int32, device="cuda"))


def prepare(case, seed):
    path = case["path"]
    if path == "run":
        run = hs.Run(_config(case, seed))
        run.step(WARM)
        out = None if run.A <= HOST_READ_AGENTS else _sample_buffers(run.A, run.SW)
        return {"case": case, "run": run, "out": out}
    if path == "clade":
        cfg = dataclasses.replace(_config(case, seed), fitness_model="tag", tournament_size=0)
        pick = torch.arange(cfg.islands, device="cuda") * cfg.pop_per_island
        return {"case": case, "cfg": cfg, "pick": pick}
    if path == "pool":
        specs = wl.c4_saved()[case["first"]:case["first"] + case["runs"]]
        cfgs = [hs.Config(**dict(s.config_kwargs(), seed=seed * 64 + s.seed)) for s in specs]
        G = 256
        need = sum((hs.footprint_bytes(c, G) + 255) & ~255 for c in cfgs)
        pool = hs.Pool(need + hs.pool_overhead_bytes(len(cfgs)) + (1 << 20), max_runs=len(cfgs),
                       max_gens_per_launch=G, block_threads=case["block"],
                       use_graph=case["graph"])
        # as long as the shortest-lived surface of the set lasts
        ids = [pool.admit(c, 131071) for c in cfgs]
        pool.advance(WARM)
        pool.sync()
        # every run's sample in slices of one buffer
        words = torch.empty(sum(c.agents * (2 + c.surface_words) for c in cfgs),
                            dtype=torch.int32, device="cuda")
        outs, at = [], 0
        for c in cfgs:
            A, SW = c.agents, c.surface_words
            outs.append((words[at:at + A], words[at + A:at + 2 * A],
                         words[at + 2 * A:at + (2 + SW) * A].view(A, SW)))
            at += (2 + SW) * A
        torch.cuda.synchronize()
        return {"case": case, "pool": pool, "runs": [pool.run(i) for i in ids], "out": outs,
                "words": words}
    if path == "serve":
        specs = wl.c5_saved()[case["first"]:case["first"] + case["requests"]]
        reqs = [dataclasses.replace(s, arrival=0.0, seed=seed * 4096 + s.seed,
                                    generations=max(1, s.generations // case["gens_div"]))
                for s in specs]
        pool = hs.Pool(SERVE_POOL_BYTES, max_runs=64, max_gens_per_launch=case["chunk"])
        return {"case": case, "pool": pool, "reqs": reqs}
    if path == "mrca":
        n = case["n"]
        run = hs.Run(_config(dict(case, w=64, h=64, n=32, tournament=2), seed))
        run.step(case["age"])
        _, cnt, srf = run.sample(n)
        lb = torch.empty((n, n), dtype=torch.int32, device="cuda")
        return {"case": case, "run": run, "cnt": cnt, "srf": srf, "lb": lb,
                "ub": torch.empty_like(lb), "ws": hs.MrcaWorkspace(case["sites"], n)}
    cnt, srf, _ = _annotations(case, seed)
    return {"case": case, "cnt": torch.from_numpy(cnt).cuda(),
            "srf": torch.from_numpy(srf).cuda()}


def run(state):
    case = state["case"]
    path = case["path"]
    if path == "run":
        r = state["run"]
        r.step(case["gens"])
        if state["out"] is None:
            box = r.outbox()
            return [x.view(np.int32) for x in r.agents() + (box or ())]
        return r.sample(r.A, out=state["out"])
    if path == "clade":
        r = hs.Run(state["cfg"])
        r.step(case["gens"])
        tags, _, _ = r.agents()
        _, cnt, srf = r.sample(r.A)
        lb, ub = r.mrca_bounds(cnt, srf)
        tree = r.phylo_tree(cnt[state["pick"]], srf[state["pick"]])
        r.close()
        return {"tags": tags.view(np.int32), "lb": lb, "ub": ub, "tree": _whole(tree)}
    if path == "pool":
        pool = state["pool"]
        pool.advance(case["gens"])
        for r, out in zip(state["runs"], state["out"]):
            r.sample(r.A, out=out)
        torch.cuda.current_stream().wait_stream(pool.stream)
        return state["words"]
    if path == "serve":
        report = srv.serve(state["pool"], state["reqs"], chunk_gens=case["chunk"],
                           sample=SERVE_SAMPLE, keep_results=True)
        return [[x.view(np.int32) for x in (r.sample_idx, r.lb, r.ub)] for r in report.results]
    if path == "mrca":
        if case["bound"]:
            return state["run"].mrca_bounds(state["cnt"], state["srf"], workspace=state["ws"],
                                            lb=state["lb"], ub=state["ub"])
        return hs.mrca_bounds(case["kind"], case["sites"], state["cnt"], state["srf"],
                              workspace=state["ws"], lb=state["lb"], ub=state["ub"],
                              bits=case["bits"], interval=case["interval"])
    return _whole(hs.phylo_tree(case["kind"], case["sites"], state["cnt"], state["srf"],
                                bits=case["bits"], interval=case["interval"]))


def _whole(tree):
    return {k: v.view(np.int32) if isinstance(v, np.ndarray) else v for k, v in tree.items()}


# ---------------------------------------------------------------------------
# What one pass cannot do without.  Operations of a birth: one Philox block
# is ten rounds of two 32x32->64 products and four XORs, and about twenty
# more pick the parent and write the child; a float birth takes two blocks
# and, for a third of the births, about a hundred binary64 steps.
OPS_INT, OPS_FLOAT = 80, 180


def _run_work(agents, islands, words, gens, ops, sampled, counter=False):
    record = 4 * (1 + words + (1 if counter else 0))
    return {"bytes": 2 * agents * record + 32 * islands + 4 * sampled * (2 + words),
            "flops": gens * agents * ops}


def work(case):
    path = case["path"]
    if path in ("run", "clade"):
        I = case["w"] * case["h"]
        A = I * case["n"]
        words = case["sites"] * case.get("bits", 1) // 32
        act = case.get("activity", 0.0)
        ops = OPS_FLOAT if case.get("model") == "float" else OPS_INT
        w = _run_work(A, I, words, case["gens"] * (act or 1.0), ops, A, bool(act))
        if path == "clade":
            w["bytes"] += 8 * A * A + 12 * I
        return w
    if path in ("pool", "serve"):
        pool = path == "pool"
        specs = (wl.c4_saved() if pool else wl.c5_saved())
        specs = specs[case["first"]:case["first"] + case["runs" if pool else "requests"]]
        total = {"bytes": 0, "flops": 0}
        for s in specs:
            gens = case["gens"] if pool else max(1, s.generations // case["gens_div"])
            n = s.agents if pool else min(SERVE_SAMPLE, s.agents)
            w = _run_work(s.agents, s.grid_w * s.grid_h, s.surface_sites // 32, gens, OPS_INT, n)
            total["bytes"] += w["bytes"] + (0 if pool else 8 * n * n)
            total["flops"] += w["flops"]
        return total
    n = case["n"]
    words = case["sites"] * case["bits"] // 32
    if path == "mrca":
        return {"bytes": 4 * n * (1 + words) + 8 * n * n, "flops": 4 * n * n}
    return {"bytes": 4 * n * (1 + words) + 12 * n,
            "flops": 2 * n * max(1, math.ceil(math.log2(n)))}


# ---------------------------------------------------------------------------
# Annotations as a population leaves them, made without the framework: the
# surface's retained deposit times from a plain replay of the site rule, and
# one resampling of n lineages on a line per doubling of the time between
# two of them, each followed by the fresh differentiae of that deposit.
def _replay(kind, S, items):
    """The item each site holds after `items` placements: a sub-surface fills
    in order, then an item takes the lowest site whose item has left the
    retention target (steady: multiples of 2^bitlen(u // (m-1)); tilted: the
    m // bitlen(u+1) newest items of each level ctz(t+1))."""
    def leaves(policy, m, t):
        if policy == "steady":
            return math.inf if t == 0 else max(t + 1, (m - 1) * (t & -t))
        low = (t + 1) & -(t + 1)
        c = (t + 1) // (2 * low)
        for B in range((t + 2).bit_length(), m + 1):
            u = max((c + m // B + 1) * 2 * low - low - 1, (1 << (B - 1)) - 1, t + 1)
            if u <= (1 << B) - 2:
                return u
        return math.inf

    held = np.full(S, -1, np.int64)
    gone = np.zeros(S)
    half = S // 2
    for T in range(items):
        policy, m, off, u = kind, S, 0, T
        if kind == "hybrid":
            policy, m, off, u = (("steady", half, 0, T // 2) if T % 2 == 0
                                 else ("tilted", half, half, T // 2))
        site = off + (u if u < m else int(np.argmax(gone[off:off + m] <= u)))
        held[site] = T
        gone[site] = leaves(policy, m, u)
    return held


def _annotations(case, seed):
    """(counter int32 [n], surface words int32 [n, W], layout in generations
    [S], -1 where empty)."""
    n, S, bits, interval = case["n"], case["sites"], case["bits"], case["interval"]
    items = -(-case["age"] // interval)
    held = _replay(case["kind"], S, items)
    rng = np.random.default_rng(seed)
    values = np.zeros((n, S), np.uint64)
    order = [int(k) for k in np.argsort(held) if held[k] >= 0]
    for j, k in enumerate(order):
        gap = int(held[k] - (held[order[j - 1]] if j else 0)) * interval
        for _ in range(min(12, max(1, gap.bit_length()))):
            step = np.rint(rng.normal(0.0, 1.0 + math.sqrt(gap), n)).astype(np.int64)
            values = values[(np.arange(n) + step) % n]
        values[:, k] = rng.integers(0, 1 << bits, n, dtype=np.uint64)
    per = 32 // bits
    shift = (np.arange(per) * bits).astype(np.uint64)
    words = (values.reshape(n, S // per, per) << shift).sum(axis=2).astype(np.uint32)
    layout = np.where(held >= 0, held * interval, -1)
    return np.full(n, case["age"], np.int32), words.view(np.int32), layout


def exact(case, seed):
    """Every output is a whole number that follows from the seed, but for the
    two means of a tree: mean distinctiveness (branch length over leaves) and
    mean pairwise distance (twice the mean time since the pairs' ancestors)."""
    if case["path"] != "tree":
        return None
    cnt, words, layout = _annotations(case, seed)
    n, bits, T = case["n"], case["bits"], case["age"]
    order = [int(k) for k in np.argsort(layout) if layout[k] >= 0]
    mask = (1 << bits) - 1
    rows = words.view(np.uint32)
    cols = np.stack([(rows[:, k * bits // 32] >> np.uint32(k * bits % 32)) & np.uint32(mask)
                     for k in order], axis=1)
    cols = cols[np.lexsort(cols.T[::-1])]
    differ = cols[1:] != cols[:-1]
    first = np.where(differ.any(axis=1), differ.argmax(axis=1), len(order))
    times = np.append(layout[order], T)[first].astype(np.int64)   # of the boundaries
    # the binary tree whose nodes are the boundaries, earliest time at the top
    # (equal times make edges of no length): a stack of nodes still open on
    # their right, each with its time and its left subtree's size and top
    branch, pairs, stack = 0, 0, []
    for t in [int(x) for x in times] + [-1]:
        size, top = 1, T
        while stack and stack[-1][0] >= t:
            at, left, left_top = stack.pop()
            branch += (left_top - at) + (top - at)
            pairs += (T - at) * left * size
            size, top = left + size, at
        stack.append((t, size, top))
    tree = {k: None for k in ("leaf_parent", "node_parent", "node_time", "sum_branch_length",
                              "pair_sum", "root_time", "internal_nodes", "status", "n", "T")}
    tree["mean_ed"] = branch / n
    tree["mean_pairwise_distance"] = 2.0 * pairs / (n * (n - 1) / 2.0) if n > 1 else 0.0
    return tree
