"""Integer births over line tiles (islands in a row of the population, one
generation per launch): bit for bit against the oracle for the runs that take
them (few agents to an island, one agent per thread in a large run) and for
launches of a single generation of any run, on both sides of the rule's
lines, for every fitness model and for asynchronous ticks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

P = lambda p: int(p * 2**32)          # noqa: E731


def check(orc, cfg, steps, shape=None):
    import paper_2404_10861_amd as hs
    run = hs.Run(cfg, max_gens_per_launch=16)
    run.set_resident(False)
    if shape:
        run.set_launch_shape(*shape)
    for g in steps:
        run.step(g)
    ref = orc.Run(cfg.grid_w, cfg.grid_h, cfg.pop_per_island, cfg.surface_sites, cfg.kind,
                  tournament=cfg.tournament_size, mut_thr=cfg.mut_threshold, mut_lo=cfg.mut_lo,
                  mut_hi=cfg.mut_hi, migrants=cfg.migrants_per_island, seed=cfg.seed,
                  fitness_model={"int": 0, "tag": 2}[cfg.fitness_model],
                  bits=cfg.differentia_bits, interval=cfg.ingest_interval,
                  activity=cfg.async_activity)
    ref.step(sum(steps))
    for got, want in zip(run.agents(), ref.agents()):
        assert np.array_equal(got, want)
    assert np.array_equal(run.layout(), ref.layout())
    for got, want in zip(run.outbox() or (), ref.outbox() or ()):
        assert np.array_equal(got, want)


@pytest.mark.parametrize("activity", [0.0, 0.6])
@pytest.mark.parametrize("w,h,n,sites,model,tournament", [
    (1, 1, 1, 64, "int", 2),
    (2, 1, 4, 32, "int", 0),
    (61, 43, 1, 32, "tag", 0),
    (37, 29, 2, 64, "int", 2),
    (300, 1, 4, 64, "int", 2),
    (1, 300, 3, 32, "int", 0),
    (53, 47, 4, 32, "int", 0),
    (41, 23, 32, 64, "int", 2),       # a launch of one generation only
    (19, 31, 7, 64, "int", 0),
])
def test_small_islands_and_single_generations(orc, w, h, n, sites, model, tournament, activity):
    import paper_2404_10861_amd as hs
    cfg = hs.Config(w, h, n, sites, "hybrid" if sites == 64 else "tilted", seed=w * h,
                    fitness_model=model, tournament_size=tournament,
                    async_activity=P(activity), ingest_interval=1 + n % 3)
    check(orc, cfg, (1, 2, 1, 33, 7, 1))


@pytest.mark.parametrize("w,h,n,sites,activity,shape", [
    (512, 256, 4, 64, 0.0, None),         # 0.5 M agents: line; 128 threads at most
    (1000, 660, 4, 64, 0.0, None),        # 2.64 M: two generations
    (303, 301, 33, 32, 0.0, None),        # 3.0 M, one agent per thread: line
    (301, 161, 33, 64, 0.0, None),        # 1.6 M on two-word surfaces: two generations
    (303, 301, 33, 32, 0.9, None),
    (300, 130, 33, 64, 0.9, None),
    (600, 437, 2, 32, 0.0, None),
    (900, 900, 3, 32, 0.0, (64, 1)),
    (100, 100, 32, 64, 0.0, (1024, 2)),   # more threads than a tile takes
])
def test_large_runs_on_both_sides_of_the_rule(orc, w, h, n, sites, activity, shape):
    import paper_2404_10861_amd as hs
    cfg = hs.Config(w, h, n, sites, "steady", seed=n, tournament_size=2,
                    async_activity=P(activity))
    check(orc, cfg, (3, 4), shape)


def test_pool_advanced_one_by_one(orc):
    """A pool's advances of one generation (line tiles, if every run has
    migration) between longer ones."""
    import paper_2404_10861_amd as hs
    cfgs = [hs.Config(13, 10, 32, 64, "tilted", seed=1, tournament_size=2),
            hs.Config(45, 7, 3, 32, "steady", seed=2, tournament_size=0),
            hs.Config(9, 9, 6, 64, "hybrid", seed=3, fitness_model="float", tournament_size=5,
                      del_threshold=P(0.33), ben_threshold=P(0.03)),
            hs.Config(8, 5, 32, 32, "tilted", seed=4, migrants_per_island=0, tournament_size=2)]
    for n in (3, 4):
        need = sum((hs.footprint_bytes(c, 8) + 255) & ~255 for c in cfgs[:n])
        pool = hs.Pool(need + hs.pool_overhead_bytes(n) + (1 << 20), max_runs=n,
                       max_gens_per_launch=8, block_threads=128)
        ids = [pool.admit(c, 1000) for c in cfgs[:n]]
        for g in (1, 1, 3, 1, 8, 1, 1, 1):
            pool.advance(g)
        pool.sync()
        for i, cfg in zip(ids, cfgs):
            ref = orc.Run(cfg.grid_w, cfg.grid_h, cfg.pop_per_island, cfg.surface_sites, cfg.kind,
                          tournament=cfg.tournament_size, mut_thr=cfg.mut_threshold,
                          mut_lo=cfg.mut_lo, mut_hi=cfg.mut_hi, migrants=cfg.migrants_per_island,
                          seed=cfg.seed, fitness_model={"int": 0, "float": 1}[cfg.fitness_model],
                          del_thr=cfg.del_threshold, ben_thr=cfg.ben_threshold,
                          del_sigma=cfg.del_sigma, ben_sigma=cfg.ben_sigma)
            ref.step(17)
            run = pool.run(i)
            for got, want in zip(run.agents(), ref.agents()):
                assert np.array_equal(got, want)
            for got, want in zip(run.outbox() or (), ref.outbox() or ()):
                assert np.array_equal(got, want)
