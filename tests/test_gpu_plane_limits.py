"""2-D fast summation jobs on both sides of the limits of the one-launch transform, against the FP64
oracle."""
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


@pytest.mark.parametrize("side", [0.5, 0.75, 1.0])
@pytest.mark.parametrize("M", [20, 27, 31, 32, 40])  # boxes of 28 to 46 cells: 300 to 1250 MFMAs
def test_tree_products(mot, side, M):
    r = rng(int(100 * side) + M)
    inst = W.make_instance(r, 3, [500, 211, 17], 2, W.TREE, 0.08, parent=W.star_parent(3))
    pts = [side * x for x in inst.points]
    fs = mot.fastsum_params(M=M, n=128, m=6, p=4, tau=1.0, eps_B=0.25)
    plan = mot.Plan(pts, inst.weights, W.TREE, inst.parent, inst.eta, path=mot.NFFT, fastsum=fs)
    for t, s in [(0, 1), (1, 0), (2, 0), (0, 2)]:
        v = r.uniform(0.0, 1.0, inst.sizes[s])
        want = oracle.kernel_apply(pts[t], pts[s], v, inst.eta)
        assert rel_to_max(plan.apply(t, s, v), want) < TOL
    plan.close()


@pytest.mark.parametrize("n0", [63, 64, 159, 160])
@pytest.mark.parametrize("n,M", [(128, 24), (128, 40), (256, 40), (256, 60)])  # 600 to 4000 MFMAs
def test_circle_rows(mot, n0, n, M):
    inst = W.make_instance(rng(n0 + M), 3, [n0, 70, 90], 2, W.CIRCLE, 0.05)
    fs = mot.fastsum_params(M=M, n=n, m=5, p=4, tau=1.0, eps_B=0.25)
    plan = mot.Plan(inst.points, inst.weights, W.CIRCLE, None, inst.eta, path=mot.NFFT, fastsum=fs)
    P, _ = plan.marginals()
    for a, b in zip(P, oracle.circle_marginals(inst.points, inst.eta, [np.ones(x) for x in inst.sizes])):
        assert rel_to_max(a, b) < 1e-5
    plan.close()


@pytest.mark.parametrize("n", [64, 128])  # boxes of about 900 and 2000 cells, folded by the transform and before it
@pytest.mark.parametrize("m", [7, 8])     # tiles of 3 and 1 cells
@pytest.mark.parametrize("chunk", [0, 8])
def test_narrow_tiles(mot, n, m, chunk):
    r = rng(n + m)
    inst = W.make_instance(r, 3, [900, 411, 17], 2, W.TREE, 0.08, parent=W.star_parent(3))
    fs = mot.fastsum_params(M=16, n=n, m=m, p=4, tau=1.0, eps_B=0.25, chunk=chunk)
    plan = mot.Plan(inst.points, inst.weights, W.TREE, inst.parent, inst.eta, path=mot.NFFT, fastsum=fs)
    assert chunk or plan.info()["chunk"] == 2048
    for t, s in [(0, 1), (1, 0), (2, 0), (0, 2)]:
        v = r.uniform(0.0, 1.0, inst.sizes[s])
        want = oracle.kernel_apply(inst.points[t], inst.points[s], v, inst.eta)
        assert rel_to_max(plan.apply(t, s, v), want) < TOL
    plan.close()
