"""The footprint of circles on the fast summation against the memory their plans hold."""
import numpy as np
import pytest

from paper_2208_03120_amd import workloads as W

pytestmark = pytest.mark.gpu


def held_and_footprint(sizes, d, eta):
    from paper_2208_03120_amd import mot
    inst = W.make_instance(np.random.Generator(np.random.PCG64(5)), len(sizes), sizes, d, W.CIRCLE, eta)
    plan = mot.Plan(inst.points, inst.weights, W.CIRCLE, None, eta, path=mot.NFFT)
    held = plan.info()["device_bytes"]
    plan.close()
    half = max(float(np.ptp(np.concatenate(inst.points)[:, c])) / 2 for c in range(d))
    return held, mot.footprint(sizes, d, W.CIRCLE, mot.NFFT, mot.PREC_MIXED, eta, half_width=half)


@pytest.mark.parametrize("sizes,d,eta", [([3, 2, 4], 1, 0.1), ([60, 400, 20, 900], 1, 0.05), ([900, 30, 500], 2, 0.1),
                                         ([20, 1200, 700, 3, 50], 2, 0.2), ([500] * 6, 2, 0.05), ([200, 300, 250], 3, 0.3)])
def test_bounds_the_plan(sizes, d, eta):
    held, fp = held_and_footprint(sizes, d, eta)
    assert held <= fp


def test_counts_no_matrix_that_is_not_there():
    """Four marginals of 3000 points in 2-D: the matrices are six of 72 MB; all that the estimate rounds
    up (patches of empty tiles, launch items, spare table bytes) stays below half of one."""
    held, fp = held_and_footprint([3000] * 4, 2, 0.1)
    assert held <= fp < held + 3000 * 3000 * 8 // 2
