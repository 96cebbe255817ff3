"""The MRCA pairs' table kernel on the host, from its own source text (one
thread per lane, tests/pair_kernel_host.cpp): every word of the bounds
against the oracle, and the words after them unchanged, at ragged sizes and
with counters up to the last one of 32 bits, which is what the kernel gives
the columns past the end.  No GPU is needed."""
import ctypes
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
QUERY = os.path.join(os.path.dirname(HERE), "paper_2404_10861_amd", "csrc", "hsga_query.hip")
KIND = {"steady": 0, "tilted": 1, "hybrid": 2}
LAST = 0xffffffff
GUARD = 2048

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")


def kernel_text():
    src = open(QUERY).read()
    surface = re.search(r"__device__ __forceinline__ uint64_t surface64.*?\n}\n", src, re.S)
    pairs = re.search(r"constexpr uint32_t kPairTileRows.*?void mrca_general_pairs_kernel.*?\n}\n",
                      src, re.S)
    return surface.group(0) + pairs.group(0)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("pairs")
    text, so = str(tmp / "kernel.inc"), str(tmp / "pairs.so")
    with open(text, "w") as f:
        f.write(kernel_text())
    res = subprocess.run(["g++", "-std=c++20", "-O2", "-w", "-shared", "-fPIC", "-pthread",
                          f'-DPAIR_KERNEL_TEXT="{text}"', "-o", so,
                          os.path.join(HERE, "pair_kernel_host.cpp")],
                         capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr[-4000:]
    return ctypes.CDLL(so)


def annotations(orc, kind, S, counters, interval):
    """Each annotation's deposit generations in ascending order, and their sites."""
    times = np.empty((len(counters), S), np.uint32)
    sites = np.empty((len(counters), S), np.uint8)
    for a, T in enumerate(counters):
        L = orc.layout(kind, S, (int(T) + interval - 1) // interval).astype(np.uint64)
        gen = np.where(L == LAST, LAST, L * interval).astype(np.uint32)
        order = np.argsort(gen, kind="stable")
        times[a], sites[a] = gen[order], order
    return times, sites


@pytest.mark.parametrize("kind,S,bits,interval,n,last", [
    ("hybrid", 64, 1, 1, 40, ()),                       # ordinary counters
    ("hybrid", 64, 1, 1 << 22, 2, (1,)),
    ("hybrid", 64, 1, 1 << 22, 100, (99,)),             # past the end of the buffers
    ("tilted", 32, 1, 1 << 22, 257, (0, 40, 256)),      # over the rows that follow
    ("steady", 8, 8, 1 << 22, 33, (5, 32)),
])
def test_pair_kernel_on_the_host(lib, orc, kind, S, bits, interval, n, last):
    rng = np.random.default_rng(n)
    top = 400 if interval == 1 else LAST
    counters = rng.integers(0, top, size=n, dtype=np.uint64).astype(np.uint32)
    counters[list(last)] = LAST
    W = S * bits // 32
    surf = rng.integers(0, 2**32, size=(n, W), dtype=np.uint64).astype(np.uint32)
    surf[n // 2] = surf[0]
    surf[-1] = surf[0] ^ 1
    times, sites = annotations(orc, KIND[kind], S, counters, interval)
    mark = 0xa5a5a5a5
    lb, ub = (np.full(n * n + GUARD, mark, np.uint32) for _ in range(2))
    p = lambda a: ctypes.c_void_p(a.ctypes.data)        # noqa: E731
    lib.pairs(S, 3 if bits == 8 else 0, n, p(counters), p(surf), p(times), p(sites), p(lb), p(ub))
    assert (lb[n * n:] == mark).all() and (ub[n * n:] == mark).all()
    olb, oub = orc.mrca_allpairs(KIND[kind], S, counters, surf, bits=bits, interval=interval)
    assert np.array_equal(lb[:n * n].reshape(n, n), olb)
    assert np.array_equal(ub[:n * n].reshape(n, n), oub)
