"""The fp32 planner, queried through the library's testing hook (no GPU:
planning is host code): what a pass lays out fits what it is given."""
import ctypes
import random

import pytest

from paper_2404_12406_amd import _lib

FWD, DGRAD, WGRAD = 0, 1, 2


@pytest.fixture(scope="module")
def lib():
    return _lib.configure(ctypes.CDLL(_lib.LIB_PATH))


def plan(lib, pas, geom):
    o = (ctypes.c_int64 * 4)()
    assert lib.ms_testing_float_plan(pas, (ctypes.c_int32 * 13)(*geom), o) == 0, geom
    return dict(zip(("splits", "partials", "z", "given"), o))


def linear(m, k_in, n_out):
    return (m, k_in, 1, 1, n_out, 1, 1, 1, 1, 1, 1, 0, 0)


def conv(n, c, h, w, k, r, s, stride, pad):
    p, q = (h + 2 * pad[0] - r) // stride[0] + 1, (w + 2 * pad[1] - s) // stride[1] + 1
    return (n, c, h, w, k, r, s, p, q, *stride, *pad)


def _drawn(rng):
    """Odd sizes above all: filters whose element count is no multiple of four,
    reductions long enough to be split as far as the workspace goes."""
    def log(lo, hi):
        return int(round(2 ** rng.uniform(lo, hi)))
    if rng.random() < 0.5:
        return linear(log(0, 15), log(0, 11), log(0, 11))
    f, g = rng.choice([1, 2, 3, 5, 7]), rng.choice([1, 3, 4])
    h, w = log(3, 7), log(3, 7)
    return conv(log(0, 6), log(0, 8), h, w, log(0, 8), min(f, h), min(g, w), (rng.randint(1, 3), rng.randint(1, 3)),
                (rng.randint(0, 2), rng.randint(0, 2)))


def test_partials_stay_inside_the_workspace(lib):
    rng = random.Random(1)
    geoms = [linear(20612, 9, 809), linear(20039, 775, 861), conv(8, 5, 101, 99, 7, 3, 3, (1, 1), (1, 1)),
             conv(64, 3, 64, 64, 11, 3, 3, (1, 1), (1, 1))]
    geoms += [_drawn(rng) for _ in range(6000)]
    split = 0
    for g in geoms:
        for pas in (FWD, DGRAD, WGRAD):
            p = plan(lib, pas, g)
            assert p["partials"] <= p["given"], (pas, g, p)
            split += p["splits"] > 1
    assert split > 1000
