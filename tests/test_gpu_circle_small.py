"""Dense circles at the edges of the small products and of the one-launch column sums, against the
FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2208_03120_amd import workloads as W
from tests.helpers import gauge_fix, max_rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mot():
    from paper_2208_03120_amd import mot as m
    return m


# the bounds that the stated precisions hold elsewhere (gauge-fixed scalings after the sweeps)
@pytest.mark.parametrize("prec,bound", [("BF16X3", 1e-5), ("FP16", 5e-4), ("BF16", 5e-3)])
@pytest.mark.parametrize("sizes", [
    (1, 33, 64, 65),        # one tile, one with a single row, a k step beyond the wavefronts' share
    (704, 705, 300, 511),   # 121 tiles of 64 x 64 and 132: the last small product and the next form
    (1536, 40, 1537, 129),  # column sums in one launch and in two
])
def test_small_dense_circles(mot, prec, bound, sizes):
    inst = W.make_instance(np.random.Generator(np.random.PCG64(sum(sizes))), len(sizes), list(sizes), 2, W.CIRCLE, 0.1)
    ophi, oS, _, _ = oracle.circle_sinkhorn(inst.points, inst.weights, inst.eta, 5)
    plan = mot.Plan(inst.points, inst.weights, W.CIRCLE, None, inst.eta, path=mot.DENSE,
                    precision=getattr(mot, "PREC_" + prec))
    rc, done, S_last, err = plan.sinkhorn(5)
    assert done == 5
    assert max_rel(gauge_fix(plan.scalings(), inst.weights), gauge_fix(ophi, inst.weights)) < bound
    assert abs(plan.S_history()[-1] - oS[-1]) < 50 * bound * abs(oS[-1])
    plan.close()


@pytest.mark.parametrize("d,sizes", [
    (1, (10, 130, 65, 90)), (2, (10, 130, 65, 90)),   # spread row by row
    (1, (70, 40, 129, 17)), (2, (17, 130, 65, 90)),   # in groups, the last with one row
    (3, (7, 60, 33, 45)),                             # 3-D: two or three rows to an item
])
def test_fast_summation_circle_rows(mot, d, sizes):
    """Products of A diag(phi), the scaling applied where the rows are spread."""
    inst = W.make_instance(np.random.Generator(np.random.PCG64(sum(sizes))), len(sizes), list(sizes), d, W.CIRCLE, 0.1)
    ophi, oS, _, _ = oracle.circle_sinkhorn(inst.points, inst.weights, inst.eta, 5)
    plan = mot.Plan(inst.points, inst.weights, W.CIRCLE, None, inst.eta, path=mot.NFFT)
    plan.sinkhorn(5)
    # the bound that circles on this path hold elsewhere
    assert max_rel(gauge_fix(plan.scalings(), inst.weights), gauge_fix(ophi, inst.weights)) < 1e-5
    np.testing.assert_allclose(plan.S_history(), oS, rtol=1e-6)
    plan.close()
