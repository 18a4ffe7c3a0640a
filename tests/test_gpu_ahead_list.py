"""A single integral's small levels lay out the next level on the device; a
traced run and a batch have the host do it.  All three give the same bits, on
both sides of every limit: children a block writes, cubes of a tile, thresholds
per parent, parts per axis, ids above 64 bits, trees that stop early."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from common import request  # noqa: E402

pytestmark = pytest.mark.gpu


def _w(D=3, **kw):
    w = dict(integrand=5, params=[2.0 + 0.3 * i for i in range(D)] + [0.4] * D, lower=[0.0] * D, upper=[1.0] * D,
             divisions=4, samples=131, trials=3, max_depth=4, sigma_mult=1.0, seed=17, eval="fp64")
    w.update(kw)
    return w


CASES = {
    "3d": _w(),
    "fp32": _w(eval="fp32"),
    "depth1": _w(max_depth=1),
    "one_cube": _w(divisions=1),
    "sigma0": _w(sigma_mult=0.0, max_depth=2),
    "tile_full_1024_sigma0": _w(D=5, divisions=4, sigma_mult=0.0, max_depth=1),   # 1024 x 32 children: over the limit
    "4d_16384_children": _w(D=2, divisions=32, sigma_mult=0.0, max_depth=2, split=4),
    "over_a_tile": _w(D=2, divisions=33, max_depth=2),
    "per_parent": _w(scope=1),
    "split3": _w(split=3, max_depth=3),
    "split5_per_parent": _w(D=2, split=5, scope=1, max_depth=3),
    "constant": _w(integrand=6, params=[2.0], sigma_mult=0.5),
    "rtol": _w(rtol=0.02, sigma_mult=0.5),
    "truncated": _w(max_cubes_per_level=100, sigma_mult=0.5),
    "nonfinite": _w(integrand=4, params=[-2.0] * 3, divisions=2, samples=997),
    "wide_ids": dict(_w(D=6, divisions=3, sigma_mult=3.0, samples=64, max_depth=11, max_cubes_per_level=4096), integrand=3,
                     params=[900.0] * 6 + [0.37] * 6),
    "user_deep": _w(D=1, divisions=7, max_depth=15, sigma_mult=0.5),
}


@pytest.fixture(scope="module")
def z():
    from paper_1902_07916_amd import Integrator
    zi = Integrator(arena_bytes=1 << 30)
    yield zi
    zi.close()


def _bits(r):
    import numpy as np
    return (np.array([r.integral, r.std] + r.thr_per_level).tobytes(), r.cubes_per_level, r.selected_per_level,
            r.flags, r.status, r.n_samples)


@pytest.mark.parametrize("case", sorted(CASES))
def test_device_list_equals_host_list(z, case):
    w = CASES[case]
    print("ahead list:", case, flush=True)
    req = request(w)
    a = z.integrate_request(req, raise_on_error=False)
    b = z.integrate_request(req, trace=True, trace_capacity=1 << 15, raise_on_error=False)
    c = z.integrate_noalloc(req, raise_on_error=False)
    other = request(_w(seed=5))
    d, e = z.integrate_batch([req, other])
    assert _bits(a) == _bits(b) == _bits(c) == _bits(d)
    # and the other one, whose company ends before or after it
    assert _bits(z.integrate_request(other)) == _bits(e)
