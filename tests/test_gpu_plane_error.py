"""Rounding of the one-launch transforms: the spread of a product's relative errors about their
mean, over 30 problems.  The rest of a product (FP32 windows, values, spreading and
interpolation) and a radix-2 transform give 6.2e-8; contractions summed as one FP32 chain gave
7.9e-8 to 8.5e-8 on these sizes.  The bound lies between: a transform that adds no more than half
of that difference."""
import numpy as np
import pytest

import oracle
from paper_2208_03120_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eta", [0.05, 0.2, 0.3])  # bands of 12, 28 and 40
def test_spread_of_errors_2d(eta):
    from paper_2208_03120_amd import mot
    var = []
    for seed in range(30):
        r = np.random.Generator(np.random.PCG64(100 + seed))
        inst = W.make_instance(r, 2, [400, 3000], 2, W.TREE, eta, parent=[-1, 0])
        plan = mot.Plan(inst.points, inst.weights, W.TREE, inst.parent, eta, path=mot.NFFT)
        v = r.uniform(0, 1, 3000)
        want = oracle.kernel_apply(inst.points[0], inst.points[1], v, eta)
        var.append(np.var((plan.apply(0, 1, v) - want) / want))
        plan.close()
    assert np.sqrt(np.mean(var)) < 7.4e-8
