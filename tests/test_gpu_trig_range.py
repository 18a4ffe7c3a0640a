"""FP64 sine and cosine integrands on both sides of the argument size where
the kernels change from their own reduction to the library's (65536): every
per-(cube, trial) sum against the oracle's libm, results that do not depend on
which kernel a batch's company selects, and the same function in a user's
body."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from common import compare_tree, oracle_problem, request  # noqa: E402

pytestmark = pytest.mark.gpu

SIN_BODY = "real t = 0; for (int i = 0; i < D; ++i) t += x[i]; return sin(t);"
COS_BODY = "real t = (real)6.283185307179586476925286766559 * (real)p[0]; " \
           "for (int i = 0; i < D; ++i) t = fma((real)p[1 + i], x[i], t); return cos(t);"


def _sin(top, dim=2, seed=3):
    # the domain's largest argument sum is `top`
    return dict(integrand=1, params=[], lower=[top / dim - 4.0] * dim, upper=[top / dim] * dim, divisions=3,
                samples=501, trials=3, max_depth=1, sigma_mult=0.5, seed=seed, eval="fp64")


def _osc(top, dim=3, seed=4):
    # no refinement: the two sides round the phase differently (the library
    # with FMAs), by top * 2^-53 per operation, which the per-trial bound of
    # compare_tree covers and its threshold check does not
    c = [top / dim] * dim
    return dict(integrand=2, params=[0.3] + c, lower=[-1.0] * dim, upper=[1.0] * dim, divisions=2, samples=601,
                trials=4, max_depth=0, sigma_mult=0.5, seed=seed, eval="fp64")


CASES = {"sin_small": _sin(2.0), "sin_below": _sin(64000.0), "sin_across": _sin(65538.0), "sin_far": _sin(1e9),
         "sin_1d": _sin(7.0, dim=1), "sin_16d": dict(_sin(48.0, dim=16), divisions=1, max_depth=0),
         "osc_below": _osc(60000.0), "osc_across": _osc(80000.0), "osc_far": _osc(1e7)}


@pytest.fixture(scope="module")
def z():
    from paper_1902_07916_amd import Integrator
    zi = Integrator(arena_bytes=1 << 30)
    yield zi
    zi.close()


@pytest.mark.parametrize("case", sorted(CASES))
def test_tree_matches_oracle(z, orc, case):
    w = CASES[case]
    print("trig range:", case, flush=True)
    r = z.integrate(**w, trace=True)
    compare_tree(orc, w, r, 1e-9, 1e-6)
    plain = z.integrate(**w)
    # the untraced kernels give the traced ones' sums
    assert (plain.integral, plain.std, plain.cubes_per_level) == (r.integral, r.std, r.cubes_per_level)


def test_batch_company_changes_nothing(z):
    """A request whose arguments stay small gives the same bits beside one of
    the same bucket whose arguments do not."""
    ws = [_sin(2.0), _sin(1e9, seed=8), _sin(64000.0, seed=9), _osc(5.0), _osc(1e12, seed=7)]
    outs = z.integrate_batch([request(w) for w in ws])
    for w, o in zip(ws, outs):
        a = z.integrate(**w)
        assert (a.integral, a.std, a.cubes_per_level) == (o.integral, o.std, o.cubes_per_level)


@pytest.mark.parametrize("case,body", [("sin_below", SIN_BODY), ("sin_across", SIN_BODY), ("sin_far", SIN_BODY),
                                       ("osc_across", COS_BODY)])
def test_user_body_gives_the_same(z, case, body):
    import paper_1902_07916_amd as pkg
    w = CASES[case]
    uid = pkg.register_integrand(body, len(w["params"]))
    a = z.integrate(**w)
    b = z.integrate(**dict(w, integrand=uid))
    assert (a.integral, a.std, a.cubes_per_level) == (b.integral, b.std, b.cubes_per_level)


@pytest.mark.parametrize("dim,eval_", [(2, "fp32"), (7, "fp32"), (8, "fp32"), (12, "fp32"), (9, "fp64")])
def test_user_kernel_traced_and_not(z, orc, dim, eval_):
    """A user body's kernel without the sums of squares (untraced levels)
    gives the sums of the one that keeps them, which match the oracle's."""
    import paper_1902_07916_amd as pkg
    from common import FP32_TRIAL_TOL, U64
    body = "real t = 1; for (int i = 0; i < D; ++i) t += (real)p[0] * x[i]; return 1 / t;"
    uid = pkg.register_integrand(body, 1)
    orc.set_user(uid, body, 1)
    w = dict(integrand=uid, params=[0.7], lower=[0.0] * dim, upper=[1.0] * dim, divisions=2 if dim < 12 else 1,
             samples=1027, trials=3, max_depth=0, sigma_mult=1.0, seed=5, eval=eval_)
    plain = z.integrate(**w)
    r = z.integrate(**w, trace=True, trace_capacity=1 << 10)
    assert (plain.integral, plain.std) == (r.integral, r.std)
    o = orc.integrate(oracle_problem(orc, w))
    # FP64: two summation orders of 1027 values, each of D + 3 roundings
    tol = FP32_TRIAL_TOL if eval_ == "fp32" else (2 * 1027 + 2 * (dim + 3)) * U64
    assert abs(r.integral - o.integral) <= tol * abs(o.integral)
