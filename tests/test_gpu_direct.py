"""Direct products at the edges of their tiles and source ranges, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2208_03120_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mot():
    from paper_2208_03120_amd import mot as m
    return m


@pytest.mark.parametrize("eta", [0.2, 0.004])  # exponent on the FP32 and on the FP64 MFMA
@pytest.mark.parametrize("d", [1, 2, 3])
def test_mixed_direct_tiles_and_ranges(mot, d, eta):
    """Targets around the 16-wide tiles and the 256-target items, sources around the
    64-source ranges and the 256-source stages.  Every term is positive.  Its relative error
    is that of the exponent (FP32 terms up to 3 * 8, a few roundings of 2^-24 each; on the
    FP64 form one rounding of at most 2^-24 * 60), of v_exp_f32 and of an FP32 sum of 64
    terms: below 1e-5 together.  Two sweeps chain at most five products."""
    sizes = [257, 1, 15, 64, 513, 16, 1100, 65]
    rng = np.random.Generator(np.random.PCG64(40 + d))
    parent = np.array([-1, 0, 0, 0, 0, 4, 4, 6], dtype=np.int32)
    inst = W.make_instance(rng, len(sizes), sizes, d, W.TREE, eta, parent=parent)
    plan = mot.Plan(inst.points, inst.weights, W.TREE, parent, eta, path=mot.DIRECT, precision=mot.PREC_MIXED)
    for t, s in [(0, 4), (6, 0), (1, 6), (6, 1), (5, 4)]:
        v = rng.uniform(0.0, 1.0, sizes[s]) ** 4
        want = oracle.kernel_apply(inst.points[t], inst.points[s], v, eta)
        np.testing.assert_allclose(plan.apply(t, s, v), want, rtol=1e-5)
    plan.sinkhorn(2)
    ophi = oracle.tree_sinkhorn(inst.points, inst.weights, parent, eta, 2)[0]
    for a, b in zip(plan.scalings(), ophi):
        np.testing.assert_allclose(a, b, rtol=5e-5)
    plan.close()


@pytest.mark.parametrize("eta", [0.2, 0.004])
def test_mixed_direct_ranges(mot, eta):
    """Products large enough for source ranges (partial sums added by a second launch) beside
    small ones, with the bounds of the test above."""
    sizes = [9001, 4097, 1100, 65]
    rng = np.random.Generator(np.random.PCG64(50))
    inst = W.make_instance(rng, 4, sizes, 2, W.TREE, eta, parent=W.star_parent(4))
    plan = mot.Plan(inst.points, inst.weights, W.TREE, inst.parent, eta, path=mot.DIRECT, precision=mot.PREC_MIXED)
    plan.sinkhorn(2)
    ophi = oracle.tree_sinkhorn(inst.points, inst.weights, inst.parent, eta, 2)[0]
    for a, b in zip(plan.scalings(), ophi):
        np.testing.assert_allclose(a, b, rtol=5e-5)
    plan.close()


@pytest.mark.parametrize("sizes", [[1, 2, 3], [129, 255, 257], [511, 1025, 640], [1700, 1650, 90], [3100, 2049, 4100]])
def test_fp64_direct_small_and_ranges(mot, sizes):
    """FP64 products in the one-launch form with 2 to 16 targets to a block and with source
    ranges; every term is positive, so the sums agree to a few roundings per product."""
    rng = np.random.Generator(np.random.PCG64(sum(sizes)))
    inst = W.make_instance(rng, 3, sizes, 3, W.TREE, 0.05, parent=W.chain_parent(3))
    plan = mot.Plan(inst.points, inst.weights, W.TREE, inst.parent, 0.05, path=mot.DIRECT, precision=mot.PREC_FP64)
    plan.sinkhorn(3)
    ophi = oracle.tree_sinkhorn(inst.points, inst.weights, inst.parent, 0.05, 3)[0]
    for a, b in zip(plan.scalings(), ophi):
        np.testing.assert_allclose(a, b, rtol=1e-12)
    plan.close()


@pytest.mark.parametrize("eta", [1e-300, 1e-9, 1.0, 1e300])
def test_fp64_direct_extreme_exponents(mot, eta):
    """Exponents far below the FP64 range (squared distances up to overflow) and at zero:
    terms are v_j at distance 0, zero where exp underflows and v_j where eta is huge."""
    x = np.array([[0.0], [1.0], [-3e-5], [1e200]])
    w = np.full(4, 0.25)
    plan = mot.Plan([x, x], [w, w], W.TREE, np.array([-1, 0], np.int32), eta, path=mot.DIRECT,
                    precision=mot.PREC_FP64)
    v = np.array([1.0, 2.0, 4.0, 8.0])
    with np.errstate(over="ignore", under="ignore"):
        d2 = (x - x.T) ** 2
        want = np.exp(-d2 / eta) @ v
    np.testing.assert_allclose(plan.apply(0, 1, v), want, rtol=1e-14)
    plan.close()
