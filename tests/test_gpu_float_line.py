"""Float births with migration over line tiles (islands in a row of the
population, one generation per launch): bit for bit against the oracle where
tiles straddle the torus's rows, end ragged, hold one island or more islands
than half their threads, on sides of 1 and 2, for synchronous runs,
asynchronous ticks, and in pools beside integer runs of two generations a
launch."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

P = lambda p: int(p * 2**32)          # noqa: E731
FLOAT = dict(fitness_model="float", tournament_size=5, del_threshold=P(0.33),
             ben_threshold=P(0.03))


def same(run, orc, cfg, gens):
    model = {"int": 0, "float": 1, "tag": 2}[cfg.fitness_model]
    ref = orc.Run(cfg.grid_w, cfg.grid_h, cfg.pop_per_island, cfg.surface_sites, cfg.kind,
                  tournament=cfg.tournament_size, mut_thr=cfg.mut_threshold, mut_lo=cfg.mut_lo,
                  mut_hi=cfg.mut_hi, migrants=cfg.migrants_per_island, seed=cfg.seed,
                  fitness_model=model, del_thr=cfg.del_threshold, ben_thr=cfg.ben_threshold,
                  del_sigma=cfg.del_sigma, ben_sigma=cfg.ben_sigma,
                  bits=cfg.differentia_bits, interval=cfg.ingest_interval,
                  activity=cfg.async_activity)
    ref.step(gens)
    for got, want in zip(run.agents(), ref.agents()):
        assert np.array_equal(got, want)
    for got, want in zip(run.outbox() or (), ref.outbox() or ()):
        assert np.array_equal(got, want)


@pytest.mark.parametrize("activity", [0.0, 0.7])
@pytest.mark.parametrize("w,h,n,sites,block,apt", [
    (1, 1, 64, 64, 64, 4),        # its own neighbour on every side
    (2, 1, 5, 32, 64, 1),
    (1, 300, 4, 64, 64, 4),       # as many islands to a tile as threads
    (23, 31, 1, 32, 128, 1),
    (17, 29, 2, 64, 256, 2),
    (45, 7, 3, 64, 256, 1),
    (37, 11, 33, 32, 64, 1),      # one island to a tile, 31 threads idle
    (29, 13, 32, 64, 256, 4),     # 32 islands to a tile
])
def test_line_tiles_match_oracle(orc, w, h, n, sites, block, apt, activity):
    import paper_2404_10861_amd as hs
    cfg = hs.Config(w, h, n, sites, "tilted", seed=w + h, async_activity=P(activity), **FLOAT)
    run = hs.Run(cfg, max_gens_per_launch=32)
    run.set_resident(False)
    run.set_launch_shape(block, apt)
    for g in (1, 2, 40):
        run.step(g)
    same(run, orc, cfg, 43)


@pytest.mark.parametrize("block,graph", [(64, False), (256, True)])
def test_pool_of_float_and_integer_runs(orc, block, graph):
    import paper_2404_10861_amd as hs
    cfgs = [hs.Config(13, 10, 32, 64, "tilted", seed=1, **FLOAT),
            hs.Config(45, 7, 16, 64, "hybrid", seed=2, tournament_size=2),
            hs.Config(9, 9, 3, 32, "steady", seed=3, **FLOAT),
            hs.Config(8, 3, 32, 32, "tilted", seed=4, migrants_per_island=0, **FLOAT)]
    need = sum((hs.footprint_bytes(c, 16) + 255) & ~255 for c in cfgs)
    pool = hs.Pool(need + hs.pool_overhead_bytes(len(cfgs)) + (1 << 20), max_runs=len(cfgs),
                   max_gens_per_launch=16, block_threads=block, use_graph=graph)
    ids = [pool.admit(c, 1000) for c in cfgs]
    for g in (1, 5, 16, 7, 16):
        pool.advance(g)
    pool.sync()
    for i, c in zip(ids, cfgs):
        same(pool.run(i), orc, c, 45)
