"""Cells of FP64 truncated plans: clouds wider in some dimensions than in others, and cubes."""
import numpy as np
import pytest

import oracle
from paper_2208_03120_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,eta,thin,cells", [
    (2, 9751, 9e-4, 0.1, 30), (2, 4516, 6e-3, 0.1, 3), (3, 3924, 2e-3, 1.0, 6), (3, 13565, 8e-4, 1.0, 8)])
def test_fp64_cells(d, n, eta, thin, cells):
    from paper_2208_03120_amd import mot
    r = np.random.Generator(np.random.PCG64(n))
    pts = [np.asfortranarray(r.uniform(-0.25, 0.25, (n, d))) for _ in range(2)]
    for x in pts:
        x[0], x[1] = -0.25, 0.25
        x[:, 0] *= thin
    pts = [np.ascontiguousarray(x) for x in pts]
    wts = [np.full(n, 1.0 / n) for _ in range(2)]
    plan = mot.Plan(pts, wts, W.TREE, [-1, 0], eta, path=mot.TRUNC, precision=mot.PREC_FP64)
    assert abs(plan.info()["n"] - cells) <= 1  # r_c and the cloud's extent set it within one
    v = r.uniform(0.5, 1.5, n)
    got, want = plan.apply(0, 1, v), oracle.kernel_apply(pts[0], pts[1], v, eta)
    plan.close()
    assert np.all(got <= want * (1 + 1e-12))
    assert np.all(got >= want * (1 - 1e-7))  # the cutoff's target
