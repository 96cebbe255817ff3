"""All-pairs MRCA bounds of annotations of different ages, bit for bit against
the oracle, on both sides of each line between the two pair kernels (the merge
of sorted time lists and the per-row tables), and byte differentiae in sizes
that take the tables: up to 4 sites always merge, 8 sites below 3,072
annotations, 32 sites below 768, 64 sites never."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KIND = {"steady": 0, "tilted": 1, "hybrid": 2}


@pytest.mark.parametrize("kind,S,bits,interval,n,ages", [
    ("steady", 8, 8, 1, 3071, 900),       # merge
    ("steady", 8, 8, 3, 3072, 900),       # tables, bytes
    ("tilted", 8, 8, 2, 3089, 200),       # tables, bytes, a ragged row tile
    ("hybrid", 8, 8, 4, 3072, 100),       # tables, bytes
    ("tilted", 32, 1, 1, 511, 3000),      # merge
    ("steady", 32, 1, 3, 512, 3000),      # merge
    ("hybrid", 32, 1, 1, 767, 900),       # merge
    ("hybrid", 32, 1, 1, 768, 900),       # tables
    ("tilted", 32, 1, 1, 1025, 3),        # tables, nearly every counter shared
    ("tilted", 64, 1, 2, 255, 3),         # tables, nearly every counter shared
    ("hybrid", 64, 1, 1, 2, 40),          # tables
    ("steady", 4, 8, 1, 3100, 60),        # merge
])
def test_pair_routes_match_oracle(orc, kind, S, bits, interval, n, ages):
    import torch
    import paper_2404_10861_amd as hs
    rng = np.random.default_rng(S * n + interval)
    counters = rng.integers(0, ages, size=n).astype(np.uint32)
    counters[0], counters[-1] = 0, ages
    W = S * bits // 32
    surf = rng.integers(0, 2**32, size=(n, W), dtype=np.uint64).astype(np.uint32)
    near = rng.random(n) < 0.5           # half of them a few bits from one surface
    surf[near] = surf[1] ^ (1 << rng.integers(0, 32, size=(int(near.sum()), W))).astype(np.uint32)
    surf[n // 2:n // 2 + 5] = surf[1]
    lb, ub = hs.mrca_bounds(kind, S, torch.from_numpy(counters.view(np.int32)).cuda(),
                            torch.from_numpy(surf.view(np.int32)).cuda(), bits=bits,
                            interval=interval)
    olb, oub = orc.mrca_allpairs(KIND[kind], S, counters, surf, bits=bits, interval=interval)
    assert np.array_equal(hs.as_u32(lb), olb) and np.array_equal(hs.as_u32(ub), oub)
