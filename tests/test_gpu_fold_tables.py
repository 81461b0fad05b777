"""Folds of 3-D boxes whose tile table does not fit in LDS, with absent, single and several chunks
to a tile, against the FP64 oracle."""
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


@pytest.mark.parametrize("m", [5, 6])  # tiles of 7 and 5 cells: covers of 3 and 4
@pytest.mark.parametrize("K", [2, 3])  # one job a launch down and up, and two
def test_table_in_global_memory(mot, m, K):
    r = np.random.Generator(np.random.PCG64(m))
    inst = W.make_instance(r, K, [900, 1100, 500][:K], 3, W.TREE, 0.06, parent=W.star_parent(K))
    pts = [np.array(x) for x in inst.points]
    for x in pts:
        x[: len(x) // 2] = 0.1 + x[: len(x) // 2] / 16  # a cluster: tiles of many chunks
    fs = mot.fastsum_params(M=32, n=512, m=m, p=4, tau=1.25, eps_B=0.25, chunk=8)
    plan = mot.Plan(pts, inst.weights, W.TREE, inst.parent, inst.eta, path=mot.NFFT, fastsum=fs)
    info = plan.info()
    assert np.prod([(L - 16) // info["tile"] + 1 for L in info["box_len"]]) >= 2048  # and one entry more
    for t, s in [(0, 1), (1, 0), (K - 1, 0), (0, K - 1)]:
        v = r.uniform(0.0, 1.0, inst.sizes[s])
        want = oracle.kernel_apply(pts[t], pts[s], v, inst.eta)
        assert rel_to_max(plan.apply(t, s, v), want) < TOL
    plan.sinkhorn(2)
    assert all(np.isfinite(x).all() for x in plan.scalings())
    plan.close()
