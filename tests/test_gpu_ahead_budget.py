"""A next level laid out ahead takes no more of the arena than one the host
lays out: a tree whose worst case just fits the static scratch, and that
reaches it, runs there.  Its root level could by sigma_mult alone be followed
by 11520 cubes; the level cap (which the reservation counts with) and the tree
stop at 256."""
import os
import re
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from common import request  # noqa: E402

pytestmark = pytest.mark.gpu

CHUNK = 8192  # points of one sampling unit: 16 bytes of partial sums each


def _w(samples, **kw):
    # a peak at a corner of the root grid: its four cubes and no other split
    w = dict(integrand=0, params=[0.004, 1.0, 7.0 / 15.0, 7.0 / 15.0], lower=[0.0] * 2, upper=[1.0] * 2, divisions=15,
             samples=samples, trials=3, max_depth=1, sigma_mult=0.5, split=8, max_cubes_per_level=256, seed=5,
             eval="fp32")
    w.update(kw)
    return w


def test_tree_that_just_fits():
    from paper_1902_07916_amd import F_TRUNCATED, Integrator, ZmcError
    z = Integrator(arena_bytes=1 << 30)
    try:
        with pytest.raises(ZmcError) as e:
            z.integrate_noalloc(request(_w(1 << 30)))
        need, holds = (int(v) for v in re.search(r"needs (\d+) bytes.*holds (\d+)", str(e.value)).groups())
        chunks = 2
        while z.request_bytes(request(_w(2 * chunks * CHUNK))) <= holds:
            chunks *= 2
        step = chunks // 2
        while step:
            if z.request_bytes(request(_w((chunks + step) * CHUNK))) <= holds:
                chunks += step
            step //= 2
        req = request(_w(chunks * CHUNK))
        spare = holds - z.request_bytes(req)
        assert 0 <= spare < 256 * 3 * 16 + 256  # one chunk's partial sums and a rounding
        print("ahead budget: spare", spare, "chunks", chunks, flush=True)
        plenty = z.integrate_request(req)
        assert plenty.cubes_per_level == [225, 256] and not plenty.flags & F_TRUNCATED
        r = z.integrate_noalloc(req)
        assert (r.integral, r.std, r.cubes_per_level) == (plenty.integral, plenty.std, plenty.cubes_per_level)
    finally:
        z.close()
