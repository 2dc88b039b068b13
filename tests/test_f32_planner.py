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
    o = (ctypes.c_int64 * 5)()
    assert lib.ms_testing_float_plan(pas, (ctypes.c_int32 * 13)(*geom), o) == 0, geom
    return dict(zip(("splits", "partials", "z", "few", "given"), o))


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


def square(c, k, s, n, f=3, stride=1):
    return conv(n, c, s, s, k, f, f, (stride, stride), (f // 2, f // 2))


# (pass, layer, whether the few-channel kernels were the faster ones by a fifth or more)
FASTER = [
    # a Linear is N images of one pixel: its tiles would hold one lane of 256
    (FWD, linear(16384, 768, 10), 0), (FWD, linear(65536, 64, 1), 0), (FWD, linear(16384, 16, 16), 0),
    (DGRAD, linear(16384, 16, 16), 0), (DGRAD, linear(1 << 25, 4, 4), 0), (FWD, linear(1 << 25, 4, 4), 0),
    # small images leave lanes without a pixel, the more they cost the more groups of channels
    (FWD, square(8, 8, 1, 60000), 0), (FWD, square(4, 4, 4, 25000), 0), (FWD, square(4, 4, 14, 2040), 1),
    (DGRAD, square(2, 2, 10, 4000), 1), (FWD, square(8, 8, 10, 4000), 0), (FWD, square(8, 8, 20, 1000), 1),
    (FWD, square(16, 16, 16, 1562), 0), (DGRAD, square(16, 16, 24, 694), 1),
    # chunks of a few channels out of wide pixels fetch every line again
    (FWD, square(64, 4, 56, 127, f=1), 0), (FWD, square(256, 4, 14, 2040, f=1), 0), (FWD, square(64, 16, 56, 24), 0),
    (FWD, square(8, 8, 56, 127, f=1), 1), (FWD, square(64, 4, 64, 64), 1),
    # few pixels
    (FWD, square(16, 16, 64, 16), 0), (FWD, square(16, 16, 64, 128), 1), (FWD, square(8, 8, 64, 32), 1),
    (DGRAD, square(3, 64, 224, 4, f=7, stride=2), 1), (DGRAD, square(3, 64, 32, 16, f=7, stride=2), 0),
    (DGRAD, square(16, 32, 64, 16, stride=2), 0),
    # the weight gradient
    (WGRAD, square(4, 4, 2, 25000), 0), (WGRAD, square(4, 4, 4, 25000), 1), (WGRAD, square(8, 8, 4, 6250), 0),
    (WGRAD, square(8, 8, 7, 8163), 1), (WGRAD, square(16, 16, 7, 8163), 0), (WGRAD, square(16, 16, 14, 2040), 1),
    (WGRAD, square(16, 16, 64, 8), 0), (WGRAD, square(16, 16, 64, 32), 1), (WGRAD, square(8, 8, 256, 64), 1),
]


@pytest.mark.parametrize("pas,geom,few", FASTER)
def test_few_channel_kernels_where_they_were_faster(lib, pas, geom, few):
    assert plan(lib, pas, geom)["few"] == few
