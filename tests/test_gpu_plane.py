"""One-launch transforms of 1-D and 2-D fast summation jobs, and the fold's covers, against the
FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2208_03120_amd import workloads as W
from tests.helpers import rel_to_max

pytestmark = pytest.mark.gpu

TOL = 2e-6  # a product's FP32 level (4e-7) and the window's own error at the cutoffs used here


@pytest.fixture(scope="module")
def mot():
    from paper_2208_03120_amd import mot as m
    return m


def rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


@pytest.mark.parametrize("d,M,n,m", [
    (1, 14, 64, 6), (1, 32, 128, 5), (1, 64, 256, 5), (1, 127, 512, 5),
    (2, 14, 64, 6),    # one launch, one tile of frequencies
    (2, 16, 64, 5),    # one launch, M + 1 = 17 frequencies: a second tile with one of them
    (2, 24, 128, 5),   # one launch, close to the limit of a tree's job
    (2, 64, 256, 5),   # the pass chain
])
@pytest.mark.parametrize("chunk", [0, 8])
def test_products_over_boxes_and_bands(mot, d, M, n, m, chunk):
    r = rng(10 * M + m)
    inst = W.make_instance(r, 3, [900, 411, 17], d, W.TREE, 0.06, parent=W.star_parent(3))
    fs = mot.fastsum_params(M=M, n=n, m=m, p=4, tau=1.0, eps_B=0.25, chunk=chunk)
    plan = mot.Plan(inst.points, inst.weights, W.TREE, inst.parent, inst.eta, path=mot.NFFT, fastsum=fs)
    for t, s in [(0, 1), (1, 0), (2, 0), (0, 2)]:
        v = r.uniform(0.0, 1.0, inst.sizes[s])
        want = oracle.kernel_apply(inst.points[t], inst.points[s], v, inst.eta)
        assert rel_to_max(plan.apply(t, s, v), want) < TOL
    plan.close()


@pytest.mark.parametrize("d", [1, 2, 3])
@pytest.mark.parametrize("m", [4, 5, 6, 7, 8])  # tiles of 9, 7, 5, 3 and 1 cells: covers 2, 3, 4 and any
def test_fold_covers(mot, d, m):
    r = rng(m)
    inst = W.make_instance(r, 2, [700, 300], d, W.TREE, 0.08)
    fs = mot.fastsum_params(M=16, n=64, m=m, p=4, tau=1.25, eps_B=0.25, chunk=16)  # 3-D clouds too
    plan = mot.Plan(inst.points, inst.weights, W.TREE, inst.parent, inst.eta, path=mot.NFFT, fastsum=fs)
    v = r.uniform(0.0, 1.0, 300)
    want = oracle.kernel_apply(inst.points[0], inst.points[1], v, inst.eta)
    assert rel_to_max(plan.apply(0, 1, v), want) < (2e-5 if m == 4 else TOL)
    plan.close()


@pytest.mark.parametrize("d,eta,N", [(2, 0.002, 70), (2, 0.1, 600), (1, 0.05, 129)])
def test_circle_rows(mot, d, eta, N):
    """Row-by-row circles, whose jobs take the one-launch transform whatever their size (the
    first one's box and spectra need more than 64 KB of LDS) and with 512 rows and more fold
    inside it."""
    inst = W.make_instance(rng(N), 3, N, d, W.CIRCLE, eta)
    plan = mot.Plan(inst.points, inst.weights, W.CIRCLE, None, eta, path=mot.NFFT)
    if eta > 0.01:
        plan.sinkhorn(2)
        ophi = oracle.circle_sinkhorn(inst.points, inst.weights, eta, 2)[0]
        for a, b in zip(plan.scalings(), ophi):
            np.testing.assert_allclose(a, b, rtol=1e-5)
    else:  # few points this far apart: compare the reduced products
        P, _ = plan.marginals()
        oP = oracle.circle_marginals(inst.points, eta, [np.ones(N)] * 3)
        for a, b in zip(P, oP):
            assert rel_to_max(a, b) < 1e-5
    plan.close()


@pytest.mark.parametrize("K", [2, 6])  # 3-D fold launches of about 300 and 1600 items: split cells and whole ones
@pytest.mark.parametrize("m", [4, 6, 8])
def test_fold_of_few_and_many_jobs(mot, K, m):
    r = rng(m + K)
    inst = W.make_instance(r, K, [600] + [500] * (K - 1), 3, W.TREE, 0.08, parent=W.star_parent(K))
    fs = mot.fastsum_params(M=16, n=64, m=m, p=4, tau=1.25, eps_B=0.25, chunk=16)
    plan = mot.Plan(inst.points, inst.weights, W.TREE, inst.parent, inst.eta, path=mot.NFFT, fastsum=fs)
    ophi, oS, _, _ = oracle.tree_sinkhorn(inst.points, inst.weights, inst.parent, inst.eta, 2)
    plan.sinkhorn(2)
    # a product's error is relative to its largest value, a corner's is an eighth of that or less,
    # and the root divides by five products of each sweep
    tol = 100 * (2e-5 if m == 4 else TOL)
    for a, b in zip(plan.scalings(), ophi):
        np.testing.assert_allclose(a, b, rtol=tol)
    plan.close()
