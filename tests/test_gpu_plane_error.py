"""Rounding of the one-launch transforms in 2-D, over 60 problems: the spread of a product's relative
errors about their mean, and how far that mean varies between problems (which two products
of an edge do not share, so that scalings drift by it in every sweep).

The rest of a product (FP32 windows, values, spreading and interpolation) and radix-2 lines give
6.2e-8 and 2.7e-8; contractions that are one FP32 chain, low frequencies first, gave 7.9e-8 to
8.5e-8 and 5e-8 on these sizes.  The bounds lie half way."""
import numpy as np
import pytest

import oracle
from paper_2208_03120_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eta", [0.05, 0.2, 0.3])  # bands of 12, 28 and 40
def test_errors_of_products_2d(eta):
    from paper_2208_03120_amd import mot
    var, mean = [], []
    for seed in range(60):
        r = np.random.Generator(np.random.PCG64(100 + seed))
        inst = W.make_instance(r, 2, [400, 3000], 2, W.TREE, eta, parent=[-1, 0])
        plan = mot.Plan(inst.points, inst.weights, W.TREE, inst.parent, inst.eta, path=mot.NFFT)
        v = r.uniform(0, 1, 3000)
        want = oracle.kernel_apply(inst.points[0], inst.points[1], v, eta)
        err = (plan.apply(0, 1, v) - want) / want
        var.append(np.var(err))
        mean.append(np.mean(err))
        plan.close()
    assert np.sqrt(np.mean(var)) < 7.4e-8
    assert np.std(mean) < 3.9e-8
