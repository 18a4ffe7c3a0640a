"""Synchronous calls that change stream from one to the next share one arena
(and the static scratch): a call ends only when nothing of it is still being
written, so the next one, on another stream, gives bitwise what it gives alone.
Trees on every route of the level kernels: one tile with the next level laid
out ahead, several tiles (the counted and the separate per-segment steps),
thresholds per parent, a tree that stops early."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from common import request  # noqa: E402

pytestmark = pytest.mark.gpu


def _w(D, divisions, seed, **kw):
    w = dict(integrand=5, params=[2.0 + 0.3 * i for i in range(D)] + [0.4] * D, lower=[0.0] * D, upper=[1.0] * D,
             divisions=divisions, samples=67, trials=3, max_depth=2, sigma_mult=1.0, seed=seed, eval="fp64")
    w.update(kw)
    return w


WORKLOADS = [_w(3, 4, 1), _w(3, 50, 2), _w(2, 600, 3, max_depth=1), _w(3, 12, 4, scope=1), _w(3, 8, 5, rtol=0.5),
             _w(2, 300, 6, max_depth=0), _w(3, 4, 7, max_depth=4)]


def _bits(r):
    import numpy as np
    return (np.array([r.integral, r.std] + r.thr_per_level).tobytes(), r.cubes_per_level, r.selected_per_level, r.flags)


def test_calls_alternating_streams():
    import torch
    from paper_1902_07916_amd import Integrator
    z = Integrator(arena_bytes=256 << 20)
    try:
        reqs = [request(w) for w in WORKLOADS]
        small = [0, 3, 4, 6]  # those that fit the static scratch
        alone = []
        for r in reqs:
            alone.append(_bits(z.integrate_request(r)))
            torch.cuda.synchronize()
        streams = [torch.cuda.Stream() for _ in range(3)]
        for k in range(60):
            i = (5 * k + k // 7) % len(reqs)
            if k % 10 == 0:
                print("streams:", k, flush=True)
            with torch.cuda.stream(streams[k % 3]):
                assert _bits(z.integrate_request(reqs[i])) == alone[i]
            j = small[k % len(small)]
            with torch.cuda.stream(streams[(k + 1) % 3]):
                assert _bits(z.integrate_noalloc(reqs[j])) == alone[j]
    finally:
        z.close()


def test_serving_stops_after_a_split():
    """Requests cancelled between the levels of a deep tree, then a stop and a
    new context on memory of the same size: the results are those of a context
    that saw no cancellation."""
    from paper_1902_07916_amd import Integrator, _abi
    deep = request(_w(3, 4, 11, max_depth=9, sigma_mult=0.3, max_cubes_per_level=1 << 14))
    ref = None
    for n in range(3):
        z = Integrator(arena_bytes=256 << 20, serve=True)
        try:
            for k in range(6):
                t = z.submit(deep)
                if n:
                    z.cancel(t)
                r = z.poll(t, wait=True)
                assert r.status in ((0, _abi.ECANCELED) if n else (0,)), r.status
            print("streams: stop", n, flush=True)
            got = _bits(z.integrate_request(deep))
            ref = ref or got
            assert got == ref
        finally:
            z.close()
