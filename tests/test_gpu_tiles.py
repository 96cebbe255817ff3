"""Launches of two generations over tiles: bit for bit against the oracle
where the tiles and the islands around them have edges -- ragged last tiles,
tori one or two islands wide or high (an island around a tile is then one of
its own, or the same on both sides), islands that cross wavefronts, tiles of
many small islands, the first generation (no emigrants yet) and odd step
counts (a launch of one generation), for each birth model, for asynchronous
ticks and without migration; and a pool of such runs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KIND = {"steady": 0, "tilted": 1, "hybrid": 2}
FLOAT = dict(fitness_model="float", tournament_size=5, del_threshold=1417339207,
             ben_threshold=128849010)
TICKS = dict(async_activity=int(0.7 * 2**32))
STEPS = (1, 2, 3, 1, 8, 17)


@pytest.fixture(scope="module")
def hs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2404_10861_amd as hs
    hs.load_library()
    return hs


def oracle_for(orc, c):
    model = {"int": 0, "float": 1, "tag": 2}[c.fitness_model]
    return orc.Run(c.grid_w, c.grid_h, c.pop_per_island, c.surface_sites,
                   KIND[c.surface_kind], tournament=c.tournament_size,
                   mut_thr=c.mut_threshold, mut_lo=c.mut_lo, mut_hi=c.mut_hi,
                   migrants=c.migrants_per_island, seed=c.seed, fitness_model=model,
                   del_thr=c.del_threshold, ben_thr=c.ben_threshold, del_sigma=c.del_sigma,
                   ben_sigma=c.ben_sigma, bits=c.differentia_bits, interval=c.ingest_interval,
                   activity=c.async_activity)


def same_state(a, b, where):
    for x, y, name in zip(a.agents(), b.agents(), ("trait", "counter", "surface")):
        assert np.array_equal(x, y), f"{name} differs {where}"
    assert np.array_equal(a.layout(), b.layout()), f"layout differs {where}"
    oa, ob = a.outbox(), b.outbox()
    assert (oa is None) == (ob is None), where
    if oa is not None:
        for x, y in zip(oa, ob):
            assert np.array_equal(x, y), f"outbox differs {where}"


@pytest.mark.parametrize("W,H,N,S,kind,extra,block", [
    (19, 13, 32, 64, "hybrid", dict(tournament_size=2), 256),
    (19, 13, 32, 64, "hybrid", dict(tournament_size=2), 64),
    (9, 5, 32, 32, "tilted", dict(tournament_size=0), 128),
    (1, 9, 32, 64, "steady", dict(tournament_size=2), 256),
    (9, 1, 32, 32, "steady", dict(tournament_size=2), 256),
    (2, 2, 32, 64, "hybrid", dict(tournament_size=2), 64),
    (1, 1, 32, 32, "tilted", dict(tournament_size=2), 64),
    (2, 11, 64, 64, "tilted", dict(tournament_size=2), 64),
    (33, 17, 1, 32, "steady", dict(tournament_size=2), 256),
    (40, 1, 1, 64, "steady", dict(tournament_size=2), 64),
    (40, 30, 1, 32, "hybrid", dict(tournament_size=0), 1024),
    (11, 9, 3, 64, "hybrid", dict(tournament_size=2), 256),
    (7, 6, 48, 64, "steady", dict(tournament_size=2), 64),
    (6, 7, 33, 32, "hybrid", dict(tournament_size=2), 256),
    (6, 7, 31, 64, "tilted", dict(tournament_size=0), 64),
    (10, 7, 16, 8, "hybrid", dict(differentia_bits=8, ingest_interval=2, tournament_size=2), 512),
    (19, 13, 32, 64, "tilted", FLOAT, 256),
    (5, 6, 17, 32, "hybrid", FLOAT, 64),
    (3, 1, 32, 64, "steady", dict(FLOAT, tournament_size=1), 64),
    (19, 13, 32, 64, "hybrid", dict(TICKS, tournament_size=2), 256),
    (1, 7, 32, 32, "steady", dict(TICKS, tournament_size=0), 64),
    (6, 7, 33, 64, "tilted", dict(TICKS, **FLOAT), 256),
    (19, 13, 32, 64, "hybrid", dict(migrants_per_island=0, tournament_size=2), 256),
    (7, 5, 31, 32, "tilted", dict(migrants_per_island=0, tournament_size=0), 64),
    (7, 5, 32, 32, "tilted", dict(TICKS, migrants_per_island=0, tournament_size=2), 64),
])
def test_tiles_match_oracle(hs, orc, W, H, N, S, kind, extra, block):
    c = hs.Config(W, H, N, S, kind, seed=11, **extra)
    run, o = hs.Run(c), oracle_for(orc, c)
    run.set_resident(False)
    run.set_launch_shape(block, 0)
    for n in STEPS:
        run.step(n)
        o.step(n)
        same_state(run, o, f"after a step of {n}")


def test_pool_of_ragged_tiles_matches_oracle(hs, orc):
    shapes = [(19, 13, 32, 64, "hybrid", 2), (1, 9, 32, 32, "steady", 2), (6, 7, 33, 64, "tilted", 0),
              (33, 17, 1, 32, "hybrid", 0), (2, 11, 64, 64, "steady", 2)]
    cfgs = [hs.Config(W, H, N, S, k, seed=20 + i, tournament_size=t)
            for i, (W, H, N, S, k, t) in enumerate(shapes)]
    cfgs.append(hs.Config(5, 6, 17, 32, "tilted", seed=30, **FLOAT))
    for block in (64, 256):
        need = sum((hs.footprint_bytes(c, 16) + 255) & ~255 for c in cfgs)
        pool = hs.Pool(need + hs.pool_overhead_bytes(len(cfgs)) + 4096, max_runs=len(cfgs),
                       max_gens_per_launch=16, block_threads=block)
        # run i stops after 20 + i generations: an odd or an even number left
        ids = [pool.admit(c, 20 + i) for i, c in enumerate(cfgs)]
        while pool.advance(7):
            pass
        pool.sync()
        for i, (c, k) in enumerate(zip(cfgs, ids)):
            o = oracle_for(orc, c)
            o.step(20 + i)
            same_state(pool.run(k), o, f"run {i} at {block} threads")


@pytest.mark.parametrize("W,H,N,S,kind,extra", [
    # many small islands: more than 64 KiB of LDS for a resident workgroup
    (32, 28, 4, 64, "hybrid", dict(tournament_size=2)),
    (32, 32, 1, 64, "steady", FLOAT),
    (32, 32, 2, 32, "tilted", dict(tournament_size=0)),
])
def test_resident_runs_of_many_small_islands_match_oracle(hs, orc, W, H, N, S, kind, extra):
    c = hs.Config(W, H, N, S, kind, seed=12, **extra)
    run, o = hs.Run(c), oracle_for(orc, c)
    assert run.resident_threads > 0
    for n in STEPS:
        run.step(n)
        o.step(n)
        same_state(run, o, f"after a step of {n}")
