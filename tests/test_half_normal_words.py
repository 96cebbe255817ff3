"""The device's half-normal evaluation (its own text, built for the host) word
by word.  Its reciprocal square root starts from a cubic and takes three Newton
steps where the definition takes six from a line; the radius is the same to the
last bit for every one of the 2^32 radius words, of which each seventh block is
compared here (HSGA_ALL_WORDS=1: all of them, 45 seconds on eight processors).
The whole radius and the angle are compared with the oracle's for blocks of
words over the whole range.  No GPU is needed."""
import ctypes
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
DEVICE = os.path.join(ROOT, "paper_2404_10861_amd", "csrc", "hsga_device.hpp")
ORACLE = os.path.join(ROOT, "oracle", "hsga_oracle.c")
CPUS = len(os.sched_getaffinity(0))
DEFINED, RADIUS, ANGLE = 0, 1, 2

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")

ORACLE_WORDS = f'''
#include "{ORACLE}"
double oracle_radius(uint32_t w) {{ return orc_sqrt_pos(-2.0 * orc_ln_u(w)); }}
double oracle_angle(uint32_t w) {{ return orc_cos_quarter(w); }}
'''


def device_text():
    src = open(DEVICE).read()
    parts = [r"constexpr uint64_t kMantissa = [^\n]*\n", r"constexpr uint64_t kExpZero = [^\n]*\n",
             r"__constant__ double kHalfNormalSeries\[31\] = \{.*?\n\};\n",
             r"template <class Coefficients>\n__device__ __forceinline__ double half_normal_radius.*?\n\}\n",
             r"template <bool SIN, class Coefficients>\n__device__ __forceinline__ double half_normal_angle.*?\n\}\n"]
    return "".join(re.search(p, src, re.S).group(0) for p in parts)


def edited(text, *edits):
    for pattern, new in edits:
        text, n = re.subn(pattern, new, text, flags=re.S)
        assert n == 1, pattern
    return text


def build(tmp, text):
    defined = edited(device_text(),
                     (r"double rs = series_step\(.*?;\n",
                      "double rs = __builtin_fma(-0.1875, q, 1.125);\n"),
                     (r"i < 3;", "i < 6;"))
    names = {n: str(tmp / n) for n in ("device.inc", "defined.inc", "oracle.c")}
    for name, body in (("device.inc", text), ("defined.inc", defined), ("oracle.c", ORACLE_WORDS)):
        with open(names[name], "w") as f:
            f.write(body)
    so = str(tmp / "half_normal.so")
    flags = ["-O3", "-march=native", "-ffp-contract=off", "-fPIC", "-w"]
    for cmd in (["gcc", *flags, "-c", "-o", names["oracle.c"] + ".o", names["oracle.c"]],
                ["g++", "-std=c++17", *flags, "-shared", "-pthread",
                 f'-DHALF_NORMAL_TEXT="{names["device.inc"]}"',
                 f'-DDEFINED_TEXT="{names["defined.inc"]}"', "-o", so,
                 os.path.join(HERE, "half_normal_host.cpp"), names["oracle.c"] + ".o"]):
        res = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
        assert res.returncode == 0, res.stderr[-4000:]
    lib = ctypes.CDLL(so)
    lib.differing.restype = ctypes.c_uint64
    lib.differing.argtypes = [ctypes.c_int, ctypes.c_uint32, ctypes.c_uint32]
    return lib


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return build(tmp_path_factory.mktemp("half_normal"), device_text())


def test_radius_words(lib):
    assert lib.differing(DEFINED, 1 if os.environ.get("HSGA_ALL_WORDS") else 7, CPUS) == 0


@pytest.mark.parametrize("what", [RADIUS, ANGLE])
def test_against_the_oracle(lib, what):
    assert lib.differing(what, 251, CPUS) == 0


def test_two_steps_would_be_seen(tmp_path):
    lib = build(tmp_path, edited(device_text(), (r"i < 3;", "i < 2;")))
    assert lib.differing(DEFINED, 4099, CPUS) > 0
    assert lib.differing(RADIUS, 4099, CPUS) > 0
