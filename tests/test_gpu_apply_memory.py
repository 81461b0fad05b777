"""Device memory of a plan over many one-product calls."""
import numpy as np
import pytest

from paper_2208_03120_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("path,precision", [("DIRECT", "PREC_FP64"), ("DIRECT", "PREC_MIXED"), ("NFFT", "PREC_MIXED"),
                                            ("TRUNC", "PREC_MIXED")])
@pytest.mark.parametrize("allocator", ["torch", None])
def test_products_do_not_add_up(path, precision, allocator):
    from paper_2208_03120_amd import mot
    r = np.random.Generator(np.random.PCG64(9))
    inst = W.make_instance(r, 3, [300, 41, 2000], 2, W.TREE, 5e-3 if path == "TRUNC" else 0.1, parent=W.star_parent(3))
    plan = mot.Plan(inst.points, inst.weights, W.TREE, inst.parent, inst.eta, path=getattr(mot, path),
                    precision=getattr(mot, precision), allocator=allocator)
    pairs = [(0, 1), (1, 0), (2, 0), (0, 2), (1, 2)]
    v = [r.uniform(0.5, 1.5, n) for n in inst.sizes]
    first = [plan.apply(t, s, v[s]) for t, s in pairs]
    held = plan.info()["device_bytes"]
    for _ in range(400):  # what a call adds would be over the slab's spare part by then
        for (t, s), want in zip(pairs, first):
            np.testing.assert_array_equal(plan.apply(t, s, v[s]), want)
    assert plan.info()["device_bytes"] == held
    # the scalings' sweeps and the products do not disturb each other
    plan.sinkhorn(2)
    for (t, s), want in zip(pairs, first):
        np.testing.assert_array_equal(plan.apply(t, s, v[s]), want)
    plan.close()
