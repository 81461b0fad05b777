"""Mixed truncated products and sweeps in sparse clouds, where a work item's run of cells is
many kernel widths long, against the FP64 oracle.

Bounds.  A term's exponent, at most 64 in size, is rounded to FP32 once (ln 2 2^-19), v_exp_f32
errs by 2^-23 at most, the value by 2^-24, and sums of 16 terms in FP32 by 15 2^-24: 2.5e-6 of
every target's own sum, whatever the range of the source values, as each term is far above
FP32's smallest number.  Sweeps keep the path's 1e-5."""
import numpy as np
import pytest

import oracle
from paper_2208_03120_amd import workloads as W
from tests.helpers import gauge_fix, max_rel
from tests.test_gpu_trunc import cutoff

pytestmark = pytest.mark.gpu

REL = np.log(2.0) * 2.0 ** -19 + 2.0 ** -23 + 16 * 2.0 ** -24


def clouds(seed, n, d, side):
    r = np.random.Generator(np.random.PCG64(seed))
    return r, [side * (r.random((n, d)) - 0.5) for _ in range(2)], [np.full(n, 1.0 / n)] * 2


# half-diagonals of a run in units of sqrt(eta / log2(e)): 13.7, 13.8, 13.8, 12.5 (the longest
# runs), 6.8 and 2.3
@pytest.mark.parametrize("d,n,eta,side", [(3, 300, 3e-4, 0.5), (3, 700, 2e-4, 0.5), (3, 500, 1e-3, 1.0),
                                          (2, 500, 3e-4, 1.0), (3, 5000, 3e-4, 0.5), (2, 5000, 3e-4, 0.5)])
@pytest.mark.parametrize("bits", [0, 60])  # source values span 2^bits
def test_product(d, n, eta, side, bits):
    from paper_2208_03120_amd import mot
    r, pts, wts = clouds(300 + d, n, d, side)
    plan = mot.Plan(pts, wts, W.TREE, [-1, 0], eta, path=mot.TRUNC)
    _, rc = cutoff(pts, eta)
    for t, s in [(0, 1), (1, 0)]:
        v = np.exp2(-r.uniform(0, bits, n)) * r.uniform(0.5, 1.5, n)
        got = plan.apply(t, s, v)
        # every source within the cutoff is in the sum, sources beyond it may be
        assert np.all(got >= oracle.kernel_apply_truncated(pts[t], pts[s], v, eta, rc) * (1 - REL))
        assert np.all(got <= oracle.kernel_apply(pts[t], pts[s], v, eta) * (1 + REL))
    plan.close()


@pytest.mark.parametrize("d,eta,side", [(3, 1e-3, 1.0), (2, 3e-4, 1.0), (3, 3e-4, 0.5)])
def test_sweeps(d, eta, side):
    """Scaling vectors that span 2^50 to 2^80."""
    from paper_2208_03120_amd import mot
    _, pts, wts = clouds(310 + d, 500, d, side)
    plan = mot.Plan(pts, wts, W.TREE, [-1, 0], eta, path=mot.TRUNC)
    plan.sinkhorn(12)
    phi, S = plan.scalings(), plan.S_history()
    plan.close()
    ophi, oS, _, _ = oracle.tree_sinkhorn(pts, wts, [-1, 0], eta, 12)
    assert max_rel(gauge_fix(phi, wts), gauge_fix(ophi, wts)) < 1e-5
    np.testing.assert_allclose(S, oS, rtol=1e-5)


@pytest.mark.parametrize("d,n,eta", [(2, 1000, 0.5), (2, 9000, 0.03), (3, 3000, 0.1), (3, 3000, 1e-3), (1, 5000, 1e-4)])
def test_fp64_launch_shape(d, n, eta):
    """FP64 plans report a launch shape that their kernel has (one or two targets per lane), and
    their products hold the cutoff's bracket."""
    from paper_2208_03120_amd import mot
    r, pts, wts = clouds(320 + d, n, d, 0.5)
    plan = mot.Plan(pts, wts, W.TREE, [-1, 0], eta, path=mot.TRUNC, precision=mot.PREC_FP64)
    info = plan.info()
    _, rc = cutoff(pts, eta)
    v = r.uniform(0.5, 1.5, n)
    got = plan.apply(0, 1, v)
    plan.close()
    assert info["m"] in (1, 2)
    assert np.all(got >= oracle.kernel_apply_truncated(pts[0], pts[1], v, eta, rc) * (1 - 1e-12))
    assert np.all(got <= oracle.kernel_apply(pts[0], pts[1], v, eta) * (1 + 1e-12))
