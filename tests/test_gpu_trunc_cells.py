"""Cells of truncated plans, which decide how far beyond the cutoff sources are still summed: clouds
wider in some dimensions than in others, cubes, and trees with small marginals."""
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


@pytest.mark.parametrize("n,eta,cells", [(5000, 3e-4, 5), (20000, 1e-3, 10), (60000, 3e-4, 12)])
def test_mixed_cells(n, eta, cells):
    from paper_2208_03120_amd import mot
    inst = W.make_instance(np.random.Generator(np.random.PCG64(n)), 3, n, 3, W.TREE, eta, parent=W.star_parent(3))
    plan = mot.Plan(inst.points, inst.weights, W.TREE, inst.parent, eta, path=mot.TRUNC)
    assert abs(plan.info()["n"] - cells) <= 1
    plan.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_small_marginals(precision):
    """Marginals of 3 and 15 points, far from some points of the others: every sum stays positive."""
    from paper_2208_03120_amd import mot
    r = np.random.Generator(np.random.PCG64(9114))
    d, K = int(r.integers(1, 4)), int(r.integers(3, 12))
    hi = int(r.choice([200, 2000, 12000]))
    sizes = [int(np.exp(r.uniform(np.log(3), np.log(hi)))) for _ in range(K)]
    eta = float(np.exp(r.uniform(np.log(1e-3), np.log(2e-2))))
    r.integers(0, 2)
    par = np.array([-1] + [int(r.integers(0, k)) for k in range(1, K)])
    inst = W.make_instance(r, K, sizes, d, W.TREE, eta, parent=par)
    plan = mot.Plan(inst.points, inst.weights, W.TREE, par, eta, path=mot.TRUNC, precision=precision)
    assert plan.sinkhorn(4)[0] == mot.MAXITER
    assert all(np.isfinite(x).all() and (x > 0).all() for x in plan.scalings())
    plan.close()
