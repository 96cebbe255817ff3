"""All-pairs MRCA bounds with the last counter of 32 bits among annotations of
other ages: bit for bit against the oracle, and the words after the bounds
unchanged (the pair kernels' columns past the end carry that counter)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KIND = {"steady": 0, "tilted": 1, "hybrid": 2}
LAST = 0xffffffff
GUARD = 4096


@pytest.mark.parametrize("kind,S,bits,n,last", [
    ("hybrid", 64, 1, 2, (1,)),
    ("hybrid", 64, 1, 257, (0, 40, 256)),
    ("tilted", 32, 1, 515, (514,)),
    ("steady", 8, 8, 3073, (7, 3072)),
    ("steady", 8, 8, 130, (129,)),       # merged pair by pair
])
def test_last_counter_stays_in_the_bounds(orc, kind, S, bits, n, last):
    import torch
    import paper_2404_10861_amd as hs
    interval = 1 << 22
    rng = np.random.default_rng(n)
    counters = rng.integers(0, LAST, size=n, dtype=np.uint64).astype(np.uint32)
    counters[list(last)] = LAST
    surf = rng.integers(0, 2**32, size=(n, S * bits // 32), dtype=np.uint64).astype(np.uint32)
    surf[n // 2] = surf[0]
    surf[-1] = surf[0] ^ 1
    mark = 0x5a5a5a5a
    out = [torch.full((n * n + GUARD,), mark, dtype=torch.int32, device="cuda") for _ in range(2)]
    hs.mrca_bounds(kind, S, torch.from_numpy(counters.view(np.int32)).cuda(),
                   torch.from_numpy(surf.view(np.int32)).cuda(), bits=bits, interval=interval,
                   lb=out[0][:n * n].view(n, n), ub=out[1][:n * n].view(n, n))
    lb, ub = (hs.as_u32(o) for o in out)
    assert (lb[n * n:] == mark).all() and (ub[n * n:] == mark).all()
    olb, oub = orc.mrca_allpairs(KIND[kind], S, counters, surf, bits=bits, interval=interval)
    assert np.array_equal(lb[:n * n].reshape(n, n), olb)
    assert np.array_equal(ub[:n * n].reshape(n, n), oub)
