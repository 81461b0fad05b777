"""Direct and truncated products of a cloud that is tiny beside its distance from the origin, with
counts that leave places of a stage of sources empty: those must add nothing.

Bound: |exponent| < 2, formed in FP32 from terms below 2 (a few 2^-24 each), and FP32 sums of
64 terms: 2e-6 relative, as for the path's other products."""
import numpy as np
import pytest

import oracle
from paper_2208_03120_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 2, 3])
@pytest.mark.parametrize("n", [1, 100, 6000])  # the one-launch form and split source ranges
def test_far_from_the_origin(n, d):
    from paper_2208_03120_amd import mot
    r = np.random.Generator(np.random.PCG64(n + d))
    eta = 1e-48
    pts = [1e-9 + 5e-25 * r.random((m, d)) for m in (n, n + 37)]
    wts = [np.full(len(p), 1.0 / len(p)) for p in pts]
    for path in (mot.DIRECT, mot.TRUNC):
        plan = mot.Plan(pts, wts, W.TREE, [-1, 0], eta, path=path)
        for t, s in [(0, 1), (1, 0)]:
            v = r.uniform(0.5, 1.5, len(pts[s]))
            np.testing.assert_allclose(plan.apply(t, s, v), oracle.kernel_apply(pts[t], pts[s], v, eta), rtol=2e-6)
        plan.sinkhorn(2)  # the sweeps' own launch shapes
        phi = plan.scalings()
        plan.close()
        want = oracle.tree_sinkhorn(pts, wts, [-1, 0], eta, 2)[0]
        for a, b in zip(phi, want):
            np.testing.assert_allclose(a, b, rtol=1e-5)
