"""Point counts around the edges of a wave's work: a group of 4 points a lane,
a whole group of 64 lanes (256 points), a chunk of 32 such groups (8192).
Every per-(cube, trial) sum against the oracle's over the same points."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from common import compare_tree  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def z():
    from paper_1902_07916_amd import Integrator
    zi = Integrator(arena_bytes=1 << 30)
    yield zi
    zi.close()


@pytest.mark.parametrize("eval_", ["fp64", "fp32"])
@pytest.mark.parametrize("dim", [1, 3, 6, 11])
@pytest.mark.parametrize("samples", [1, 3, 4, 253, 255, 256, 257, 511, 8191, 8192, 8193, 8449])
def test_sums_match_oracle(z, orc, samples, dim, eval_):
    # the corner peak is nowhere small, so no sum is short of digits
    w = dict(integrand=4, params=[0.5 + 0.1 * i for i in range(dim)], lower=[0.0] * dim, upper=[1.0] * dim,
             divisions=2 if dim < 11 else 1, samples=samples, trials=2, max_depth=0, sigma_mult=1.0, seed=samples,
             eval=eval_)
    print("ragged groups:", samples, dim, eval_, flush=True)
    r = z.integrate(**w, trace=True, trace_capacity=1 << 7)
    compare_tree(orc, w, r, 1e-9 if eval_ == "fp64" else 1e-4, 1e-6 if eval_ == "fp64" else 1e-4)
    plain = z.integrate(**w)
    assert (plain.integral, plain.std) == (r.integral, r.std)


@pytest.mark.parametrize("dim,samples", [(2, 1027), (5, 1027), (5, 8193), (7, 1027), (7, 1022), (11, 1024), (11, 1027)])
def test_product_rounded_before_the_sum(z, dim, samples):
    """An FP32 value that ends in a product is rounded before it is added
    where points are masked and from D = 10 on: the bits of a body that rounds
    it itself."""
    import paper_1902_07916_amd as pkg
    head = "real t = 1; for (int i = 0; i < D; ++i) t += (real)p[0] * x[i]; "
    w = dict(params=[0.7], lower=[0.0] * dim, upper=[1.0] * dim, divisions=2 if dim < 11 else 1, samples=samples,
             trials=3, max_depth=0, sigma_mult=1.0, seed=7, eval="fp32")
    print("product:", dim, samples, flush=True)
    a = z.integrate(**w, integrand=pkg.register_integrand(head + "return t * x[0];", 1))
    b = z.integrate(**w, integrand=pkg.register_integrand(head + 'real v = t * x[0]; asm("" : "+v"(v)); return v;', 1))
    assert (a.integral, a.std, a.stderr) == (b.integral, b.std, b.stderr)
