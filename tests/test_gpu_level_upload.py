"""A level's tables go up through the next-list kernel or through a copy
command, by the number of integrals, of new ones and of tiles: batches on both
sides of each limit give every member the bits of its result alone."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from common import request  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def z():
    from paper_1902_07916_amd import Integrator
    zi = Integrator(arena_bytes=2 << 30, max_slots=64)
    yield zi
    zi.close()


def _w(i, **kw):
    # all of them refine twice, some to several tiles
    D = 2 + i % 3
    w = dict(integrand=5, params=[3.0 + 0.1 * i] * D + [0.4] * D, lower=[0.0] * D, upper=[1.0] * D,
             divisions=(13, 7, 4)[i % 3], samples=65 + 7 * i, trials=2 + i % 4, max_depth=2, sigma_mult=0.5,
             seed=100 + i, eval=("fp64", "fp32")[i % 2])
    w.update(kw)
    return w


def _bits(r):
    return (r.integral, r.std, r.cubes_per_level, r.selected_per_level, r.thr_per_level[:-1], r.flags, r.status)


# 8 | 9 new integrals in one launch; 17 | 18 segments fill the directly read
# table; 64 every slot
@pytest.mark.parametrize("n", [1, 8, 9, 17, 18, 64])
def test_batch_equals_alone(z, n):
    print("level upload: batch of", n, flush=True)
    ws = [_w(i) for i in range(n)]
    for w, o in zip(ws, z.integrate_batch([request(w) for w in ws])):
        assert o.levels_run == 3
        assert _bits(z.integrate(**w)) == _bits(o)


# the last level of one, and of the other, side of 256 tiles to spawn from
@pytest.mark.parametrize("divisions", [508, 516])
def test_many_tiles_beside_a_small_one(z, divisions):
    big = _w(0, divisions=divisions, max_depth=1, samples=64, trials=2)
    small = _w(1)
    a, b = z.integrate(**big), z.integrate(**small)
    assert a.cubes_per_level[0] == divisions ** 2 and a.levels_run == 2
    o = z.integrate_batch([request(big), request(small)])
    assert _bits(o[0]) == _bits(a) and _bits(o[1]) == _bits(b)


def test_level_times(z):
    """The sampling time of a level is part of its wall time, for levels the
    host watches to their end and for one it blocks for."""
    for w in (_w(0), _w(1, divisions=30, samples=20000)):
        r = z.integrate(**w)
        for s, t in zip(r.sample_ms_per_level, r.ms_per_level):
            assert 0.0 < s < t
