"""Run-time compiled kernels on both sides of what their build depends on: from
10 dimensions on a group's words are generated in two halves, and an FP32 body
of many registers is compiled a second time, with a register bound or with the
halves kept apart."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.gpu

SIN_BODY = "real t = 0; for (int i = 0; i < D; ++i) t += x[i]; return sin(t);"
# three dependent D x D products, all of whose rows the last sum needs: about
# 130 registers at D = 3
WIDE_BODY = """
real y[D], w[D], v[D];
for (int i = 0; i < D; ++i) { y[i] = 0; for (int j = 0; j < D; ++j) y[i] += x[j] * (real)(1 + (i * 7 + j * 3) % 5) * (real)p[0]; }
for (int i = 0; i < D; ++i) { w[i] = 0; for (int j = 0; j < D; ++j) w[i] += y[j] * x[(i + j) % D]; }
for (int i = 0; i < D; ++i) { v[i] = 0; for (int j = 0; j < D; ++j) v[i] += w[j] * y[(i + 2 * j) % D] + x[(i * j) % D]; }
real t = 0;
for (int i = 0; i < D; ++i) for (int j = 0; j < D; ++j) t += sqrt(w[i] * w[j] + y[i] * v[j] + x[i] + (real)100);
return t;
"""


@pytest.fixture(scope="module")
def z():
    from paper_1902_07916_amd import Integrator
    zi = Integrator(arena_bytes=1 << 30)
    yield zi
    zi.close()


@pytest.mark.parametrize("samples", [1024, 1027])
@pytest.mark.parametrize("dim", [9, 10, 11, 15, 16])
def test_halves_give_the_registrys_bits(z, dim, samples):
    import paper_1902_07916_amd as pkg
    uid = pkg.register_integrand(SIN_BODY, 0)
    print("user kernels:", dim, samples, flush=True)
    w = dict(params=[], lower=[0.0] * dim, upper=[1.0] * dim, divisions=2 if dim < 12 else 1, samples=samples,
             trials=3, max_depth=0, sigma_mult=1.0, seed=5, eval="fp64")
    a, b = z.integrate(1, **w), z.integrate(uid, **w)
    assert (a.integral, a.std) == (b.integral, b.std)


@pytest.mark.parametrize("dim", [2, 3, 8])
def test_bodies_of_many_registers(z, dim):
    """The same points in both evaluation modes: every term is positive and
    takes fewer than 12 D roundings, and the point itself one."""
    import paper_1902_07916_amd as pkg
    uid = pkg.register_integrand(WIDE_BODY, 1)
    print("user kernels: wide", dim, flush=True)
    w = dict(params=[0.3], lower=[0.0] * dim, upper=[1.0] * dim, divisions=2, samples=515,
             trials=3, max_depth=0, sigma_mult=1.0, seed=5)
    a, b = z.integrate(uid, **w, eval="fp32"), z.integrate(uid, **w, eval="fp64")
    t = z.integrate(uid, **w, eval="fp32", trace=True, trace_capacity=1 << 10)
    assert abs(a.integral - b.integral) <= (12 * dim + dim * dim) * 2.0 ** -24 * b.integral
    assert (a.integral, a.std) == (t.integral, t.std)


@pytest.mark.parametrize("samples", [1024, 1027, 200])
@pytest.mark.parametrize("dim", [11, 13])
def test_halves_kept_apart(z, dim, samples):
    """An FP32 Gaussian body, whose first build spills at 11 and 13 dimensions:
    the kept build against the FP64 estimate of the same points, and against
    the traced kernel, which is built by itself."""
    import paper_1902_07916_amd as pkg
    uid = pkg.register_integrand("real q = 0; for (int i = 0; i < D; ++i) { real d = x[i] - (real)p[1]; q += d * d; } "
                                 "return exp(-q / (real)(2 * p[0] * p[0]));", 2)
    print("user kernels: apart", dim, samples, flush=True)
    w = dict(params=[1.0, 0.4], lower=[0.0] * dim, upper=[1.0] * dim, divisions=1, samples=samples, trials=3,
             max_depth=0, sigma_mult=1.0, seed=5)
    a, b = z.integrate(uid, **w, eval="fp32"), z.integrate(uid, **w, eval="fp64")
    t = z.integrate(uid, **w, eval="fp32", trace=True, trace_capacity=16)
    # q <= 0.36 D takes D + 1 roundings in sequence and each d one, exp's argument
    # one more and exp itself a few; the group's sums two
    assert abs(a.integral - b.integral) <= (0.18 * dim * (dim + 5) + 8) * 2.0 ** -24 * b.integral
    assert (a.integral, a.std) == (t.integral, t.std)
