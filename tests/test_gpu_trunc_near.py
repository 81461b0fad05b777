"""Mixed truncated products in 1-D and 2-D on both sides of the limit of the exponents of FP32
differences, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2208_03120_amd import workloads as W

pytestmark = pytest.mark.gpu

# a scaled coordinate of up to 3 + sqrt(-log2 eps) is rounded at 2^-24 of it, its difference by twice
# that; a term of exponent -x moves by 2 sqrt(x) times as much, and terms beyond x = 12 weigh 2^-12
REL = 2 * np.sqrt(12.0) * 2 * 9 * 2.0 ** -24 * np.log(2.0) + 2.0 ** -20


def cutoff(pts, eta, target=1e-7):
    d = pts[0].shape[1]
    lo, hi = (f([f(p, axis=0) for p in pts], axis=0) for f in (np.min, np.max))
    V = np.prod(np.maximum(hi - lo, np.sqrt(np.pi * eta)))
    return target * min(1.0, (np.pi * eta) ** (0.5 * d) / (2.0 ** d * V))


# cells from a point or less (few points) to hundreds: long runs beyond the limit, single cells within
@pytest.mark.parametrize("d,eta", [(1, 1e-4), (1, 3e-3), (2, 3e-4), (2, 3e-3)])
@pytest.mark.parametrize("nt,ns", [(40, 300), (300, 40), (2000, 2000), (6000, 1), (17, 9000), (9000, 5000)])
def test_product(d, eta, nt, ns):
    from paper_2208_03120_amd import mot
    r = np.random.Generator(np.random.PCG64(d + nt + ns))
    pts = [r.uniform(-0.25, 0.25, (n, d)) for n in (nt, ns)]
    if ns > 1:  # a source near each target, so that relative errors are those of its own sum
        pts[1][: min(nt, ns)] = pts[0][: min(nt, ns)] + r.normal(0.0, np.sqrt(eta) / 4, (min(nt, ns), d))
    wts = [np.full(n, 1.0 / n) for n in (nt, ns)]
    plan = mot.Plan(pts, wts, W.TREE, [-1, 0], eta, path=mot.TRUNC, precision=mot.PREC_MIXED)
    eps = cutoff(pts, eta)
    for t, s in ((0, 1), (1, 0)):
        v = np.exp2(-r.uniform(0, 6, len(pts[s]))) * r.uniform(0.5, 1.5, len(pts[s]))
        got, want = plan.apply(t, s, v), oracle.kernel_apply(pts[t], pts[s], v, eta)
        assert np.all(np.abs(got - want) <= REL * want + eps * v.sum())
    plan.close()
