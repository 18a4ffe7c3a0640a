"""FP64 sine and cosine of the sampling kernels (csrc/zmc_trig.hpp), the header
itself compiled for the CPU: within one unit in the last place of the value for
random arguments, and correctly rounded up to a hundredth where the argument is
the double nearest a multiple of pi/2 or a neighbour of it, where all but the
last bits of the reduction cancel.  On the GPU the same arguments through a
user's body."""
import ctypes as C
import math
import os
import subprocess
import sys
from fractions import Fraction

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, HERE)
CSRC = os.path.join(os.path.dirname(HERE), "paper_1902_07916_amd", "csrc")
BUILD = os.path.join(HERE, "_build")

STUB = """
#include <math.h>
#include <stdint.h>
#include <string.h>
#define __device__ static
#define __forceinline__ inline
static inline uint64_t bits(double v) { uint64_t u; memcpy(&u, &v, 8); return u; }
static inline int __double2loint(double v) { return (int)(uint32_t)bits(v); }
static inline int __double2hiint(double v) { return (int)(uint32_t)(bits(v) >> 32); }
static inline double __hiloint2double(int h, int l)
{ uint64_t u = (uint64_t)(uint32_t)h << 32 | (uint32_t)l; double v; memcpy(&v, &u, 8); return v; }
static inline uint32_t bitop3(uint32_t a, uint32_t b, uint32_t c, int t)
{ uint32_t r = 0; for (int i = 0; i < 8; ++i) if (t >> i & 1) r |= (i & 4 ? a : ~a) & (i & 2 ? b : ~b) & (i & 1 ? c : ~c); return r; }
#define __builtin_amdgcn_bitop3_b32 bitop3
"""
MAIN = """
#include "zmc_trig.hpp"
extern "C" void run(const double* t, double* out, long n, int which)
{ for (long i = 0; i < n; ++i) out[i] = which == 0 ? zmc::sin_f64(t[i]) : which == 1 ? zmc::cos_f64(t[i])
                                      : which == 2 ? zmc::trig_reduced<0>(t[i]) : zmc::trig_reduced<1>(t[i]); }
"""

# pi/2 to 300 bits, by Machin's formula
def _arctan_inv(x, one):
    s, t, k = 0, one // x, 0
    while t:
        s += t // (2 * k + 1) if k % 2 == 0 else -(t // (2 * k + 1))
        t //= x * x
        k += 1
    return s


_ONE = 1 << 320
HALF_PI = Fraction(2 * (4 * _arctan_inv(5, _ONE) - _arctan_inv(239, _ONE)), _ONE)


@pytest.fixture(scope="module")
def trig():
    inc = os.path.join(BUILD, "trig", "hip")
    os.makedirs(inc, exist_ok=True)
    with open(os.path.join(inc, "hip_runtime.h"), "w") as f:
        f.write(STUB)
    src, lib = os.path.join(BUILD, "trig", "trig.cpp"), os.path.join(BUILD, "trig", "trig_%d.so" % os.getpid())
    with open(src, "w") as f:
        f.write(MAIN)
    # every fused operation of the header is written out; nothing else fuses
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-I" + os.path.dirname(inc),
                    "-I" + CSRC, src, "-o", lib], check=True)
    L = C.CDLL(lib)
    os.unlink(lib)

    def call(t, which):
        t = np.ascontiguousarray(t, dtype=np.float64)
        out = np.empty_like(t)
        P = C.POINTER(C.c_double)
        L.run(t.ctypes.data_as(P), out.ctypes.data_as(P), C.c_long(len(t)), which)
        return out
    return call


def _near_multiples(ns):
    """(t, n) for the double nearest n pi/2 and its neighbours."""
    out = []
    for n in ns:
        t = float(n * HALF_PI)
        for v in (math.nextafter(t, -math.inf), t, math.nextafter(t, math.inf)):
            out.append((v, n))
    return out


def _value(t, n, which):
    """sin (which = 0) or cos (1) of t, as a fraction; |t - n pi/2| is tiny."""
    r = Fraction(t) - n * HALF_PI
    q = (n + which) % 4
    v = 1 - r * r / 2 if q % 2 else r - r ** 3 / 6
    return -v if q >= 2 else v


def _ulps(got, want):
    want_f = float(want)
    return abs(float((Fraction(got) - want) / Fraction(math.ulp(want_f))))


NS = sorted(set(list(range(-40, 0)) + list(range(1, 41)) + [29, 14479, 26048] + list(range(41, 41722, 97))))


@pytest.mark.parametrize("which", [0, 1])
def test_beside_multiples_of_half_pi(trig, which):
    pts = [(t, n) for t, n in _near_multiples(NS) if abs(t) <= 65536.0]
    got = trig([t for t, _ in pts], which)
    worst = max((_ulps(g, _value(t, n, which)), t) for g, (t, n) in zip(got, pts))
    assert worst[0] < 0.51, worst


@pytest.mark.parametrize("top", [0.8, 1.6, 60.0, 65000.0])
@pytest.mark.parametrize("which", [0, 1])
def test_random_arguments(trig, which, top):
    t = np.random.default_rng(5).uniform(-top, top, 200000)
    want = (np.sin, np.cos)[which](t.astype(np.longdouble))  # 64-bit significands
    err = np.abs((trig(t, which) - want) / np.spacing(np.abs(want).astype(np.float64)))
    assert np.finfo(np.longdouble).nmant >= 63
    assert err.max() < 1.0 and math.sqrt(float((err ** 2).mean())) < 0.30


def test_edges(trig):
    tiny = np.array([5e-324, -5e-324, 1e-310, -2.0 ** -1042, 2.0 ** -1042, 1e-300, -1e-300, 1e-20])
    assert np.array_equal(trig(tiny, 0), tiny) and np.array_equal(trig(tiny, 1), np.ones(8))
    z = trig(np.array([0.0, -0.0]), 0)
    assert not np.signbit(z[0]) and np.signbit(z[1]) and (z == 0).all()
    far = np.array([65536.0, -65536.0, 65536.5, 1e22, 1e300])
    for which in (0, 1):
        want = (np.sin, np.cos)[which](far)
        assert np.abs(trig(far, which) - want).max() <= 2.0 ** -53
    assert np.isnan(trig(np.array([math.inf, -math.inf, math.nan]), 0)).all()
    # the checked form gives the unchecked one's values wherever it applies
    t = np.random.default_rng(6).uniform(-65535.0, 65535.0, 100000)
    assert np.array_equal(trig(t, 0), trig(t, 2)) and np.array_equal(trig(t, 1), trig(t, 3))


@pytest.mark.gpu
def test_user_body():
    """A constant body: the estimate is the value itself, up to the rounding
    of four additions of it (2 ulp allowed)."""
    import paper_1902_07916_amd as pkg
    z = pkg.Integrator(arena_bytes=256 << 20)
    try:
        uid = pkg.register_integrand("return p[1] > 0 ? cos(p[0]) : sin(p[0]);", 2)
        sign = pkg.register_integrand("return copysign((real)1, (real)sin(p[0]));", 1)
        print("trig accuracy: user bodies", flush=True)
        call = lambda f, p: z.integrate(f, p, [0.0], [1.0], 1, 256, 2, 0, 1.0, 1).integral  # noqa: E731
        for t, n in _near_multiples([1, 2, 29, -29, 14479, 41721]):
            for which in (0, 1):
                got = call(uid, [t, float(which)])
                assert _ulps(got, _value(t, n, which)) < 2.0, (t, which)
        assert [call(sign, [v]) for v in (0.0, -0.0, 1.0, -1.0)] == [1.0, -1.0, 1.0, -1.0]
    finally:
        z.close()
