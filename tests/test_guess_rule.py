"""When a sample's counts are trusted to select the classes of a long vector
(csrc/qdot_guess.hpp), on the host: the rule's functions are compiled for it
and fed with drawn counts of laws whose bins' shares are known.  A sum by
wrong classes is made twice, so it must be rare."""
import ctypes as C
import math
import os
import subprocess

import numpy as np
import pytest
from scipy.special import erf

import paper_2105_00115_amd as q
from paper_2105_00115_amd.build import HIPCC

CSRC = os.path.join(os.path.dirname(os.path.abspath(q.__file__)), "csrc")
SOURCE = """
#include "qdot_guess.hpp"
using namespace qd;
extern "C" int top(const unsigned int *h, int t, int up) { return top_holds(h, t, up); }
extern "C" int slot(unsigned int m, int cl, int score, int ns, int mu)
{ return slot_risk(m, cl, score, ns, mu); }
extern "C" int limit() { return GUESS_RISK; }
extern "C" int seen() { return (int)GUESS_SEEN; }
"""
PERF, HALF, SINGLE, DOUBLE = range(4)
TOLS = (1e-3, 1e-4, 1e-5, 1e-6, 1e-8, 1e-10)
SAMPLE = 1 << 22


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("guess")
    src, lib = d / "guess.hip", d / "guess.so"
    src.write_text(SOURCE)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-std=c++17",
                    "-fPIC", "-shared", "-I", CSRC,
                    "-I", os.path.join(os.path.dirname(os.path.dirname(CSRC)), "include"),
                    str(src), "-o", str(lib)], check=True)
    return C.CDLL(str(lib))


# ---- shares of the bins [2^k, 2^(k+1)), k = -60 .. 140 ----------------------
K = np.arange(-60, 141)


def _shares(cdf):
    e = cdf(2.0 ** np.arange(-60.0, 142.0))
    p = np.maximum(np.diff(e), 0.0)
    return p / p.sum()


def _loguniform(decades):
    """Product of two 10**U[-d, d]: triangular in the exponent."""
    w = 2.0 * decades * math.log2(10.0)

    def cdf(z):
        u = np.clip(np.log2(z) / w, -1.0, 1.0)
        return np.where(u < 0, 0.5 * (1 + u) ** 2, 1 - 0.5 * (1 - u) ** 2)
    return _shares(cdf)


def _uniform(z):
    z = np.minimum(z, 1.0)
    return z * (1.0 - np.log(z))


def _normal(z):
    return erf(z / math.sqrt(2.0))


def _normal_loguniform(z):
    """Normal times 10**U[-3, 3], as in pairs that cancel."""
    u = (np.arange(4000) + 0.5) / 4000 * 6.0 - 3.0
    return erf(z[:, None] / 10.0 ** u[None, :] / math.sqrt(2.0)).mean(axis=1)


LAWS = {"loguniform 20": _loguniform(20), "loguniform 12": _loguniform(12),
        "loguniform 3": _loguniform(3), "uniform": _shares(_uniform),
        "normal": _shares(_normal), "cancelling": _shares(_normal_loguniform)}


# ---- the classes (exact bins), and the guess from a sample -------------------
def _floor_log2(x):
    return math.frexp(x)[1] - 1


def _ceil_log2(m):
    return (int(m) - 1).bit_length()


def _class(sigma):
    return PERF if sigma < 0 else HALF if sigma < 10 else SINGLE if sigma < 23 else DOUBLE


def _select(h, tol, up=0):
    live = np.nonzero(h)[0]
    top, bot = int(live[-1]), int(live[0])
    t = _floor_log2(tol / live.size)
    cls = {int(j): _class(_ceil_log2(h[j]) + up + int(j) - top - t + 1) for j in live}
    return top, bot, live.size, t, cls


def _guess(rule, h, tol, up, mu_single=0):
    top, bot, bins, t, _ = _select(h, tol, up)
    if not rule.top(h.ctypes.data_as(C.POINTER(C.c_uint)), top, up):
        return False
    dense = next((j for j in range(bot, top + 1) if h[j] >= rule.seen()), len(h))
    empty = risk = 0
    for j in range(bot - 1, top + 1):
        m = int(h[j]) if j >= bot else 0
        if m == 0 and not (j < dense and bot < dense):
            continue
        empty += m == 0 and j >= bot
        risk += rule.slot(m, _ceil_log2(m) if m else 0, j - top - t + 1 + up, 0, mu_single)
    if bot < dense and _floor_log2(tol / (bins + empty + up + 2)) != t:
        return False
    return risk <= rule.limit()


@pytest.mark.parametrize("law", list(LAWS))
@pytest.mark.parametrize("up", [2, 5])
def test_guesses_rarely_fail(rule, law, up):
    """At most one call in 30 sums for nothing (180 calls per law and length:
    thirty draws, six tolerances).  The end of a log-uniform range is seen in
    every draw, so that its calls are refused for a count near a boundary
    alone."""
    g = np.random.default_rng(17)
    p = LAWS[law]
    calls = stood = missed = 0
    for _ in range(30):
        h = np.ascontiguousarray(g.multinomial(SAMPLE, p), dtype=np.uint32)
        whole = h.astype(np.int64) + g.multinomial(SAMPLE * ((1 << up) - 1), p)
        if law.startswith("loguniform"):
            assert rule.top(h.ctypes.data_as(C.POINTER(C.c_uint)), int(np.nonzero(h)[0][-1]), up)
        for tol in TOLS:
            calls += 1
            if not _guess(rule, h, tol, up):
                continue
            s, w = _select(h, tol, up), _select(whole, tol)
            right = s[0] == w[0] and s[3] == w[3] and all(
                s[4].get(j, PERF) == c for j, c in w[4].items())
            stood += right
            missed += not right
    assert missed <= calls // 30, (calls, stood, missed)
    if law.startswith("loguniform"):
        assert stood


def test_counts_near_a_power_of_two_are_risky(rule):
    one = 1 << 16
    # a count of 1000 within a power of two of 1024 by 24, standard deviation
    # 31.6: 0.22 where the next power has another class, 0 where it has not
    r = rule.slot(1000, 10, -1, 0, 0)
    assert abs(r / one - 0.5 * math.erfc(24 / math.sqrt(1001) / math.sqrt(2))) < 1e-3
    assert rule.slot(1000, 10, -5, 0, 0) == 0
    # a bin that the sample missed: only where it would be kept
    assert rule.slot(0, 0, -1, 0, 0) == 0 and rule.slot(0, 0, 0, 0, 0) == one
    # a rare one: wherever the next power of two has another class
    assert rule.slot(5, 3, -3, 0, 0) == one and rule.slot(5, 3, -7, 0, 0) == 0
    # the non-strict reading moves every boundary up by one
    assert rule.slot(1000, 10, 0, 1, 0) == r
