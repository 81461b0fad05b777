"""Batches whose plans share lanes by dimension: the same bits as plans swept alone."""
import numpy as np
import pytest

from paper_2208_03120_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [
    [2, 2, 2],             # one dimension in several lanes
    [1, 3],                # a lane each
    [3, 1, 3, 2, 3, 1],    # four lanes, two of them for 3-D
    [1, 2, 3, 1, 1, 2, 2],
])
def test_lanes_by_dimension(dims):
    from paper_2208_03120_amd import mot
    plans = []
    for twice in range(2):
        for i, d in enumerate(dims):
            r = np.random.Generator(np.random.PCG64(10 * i + d))
            K = 2 + i % 3
            inst = W.make_instance(r, K, [300 + 97 * i] * K, d, W.TREE, 0.1, parent=W.star_parent(K))
            plans.append(mot.Plan(inst.points, inst.weights, W.TREE, inst.parent, inst.eta, path=mot.NFFT))
    alone, together = plans[:len(dims)], plans[len(dims):]
    for p in alone:
        p.sinkhorn(3)
    batch = mot.Batch(together)
    batch.sinkhorn(3)
    for a, b in zip(alone, together):
        for x, y in zip(a.scalings(), b.scalings()):
            np.testing.assert_array_equal(x, y)
        np.testing.assert_array_equal(a.S_history(), b.S_history())
    batch.close()
    for p in plans:
        p.close()


@pytest.mark.parametrize("dims,sizes,lanes", [
    ([2, 3, 3], [400, 90000, 90000], [2, 3, 3]),        # no 1-D plan; the 3-D plans are worth two lanes
    ([2, 2, 3, 3], [400, 400, 90000, 90000], [2, 3, 3]),
    ([2, 2, 3, 3], [400, 400, 400, 400], [2, 3]),       # too little work for a lane more
    ([1, 1, 3], [400, 400, 180000], [1, 3]),            # most work in a dimension of one plan
])
def test_lanes_beyond_one_a_dimension(dims, sizes, lanes):
    """A lane's launches are those of one of its plans, as trees of one shape share theirs; the
    finalisation is shared by all lanes."""
    from paper_2208_03120_amd import mot
    plans, own = [], {}
    for i, (d, n) in enumerate(zip(dims, sizes)):
        inst = W.make_instance(np.random.Generator(np.random.PCG64(i)), 3, [n] * 3, d, W.TREE, 0.1,
                               parent=W.star_parent(3))
        plans.append(mot.Plan(inst.points, inst.weights, W.TREE, inst.parent, inst.eta, path=mot.NFFT))
        alone = mot.Batch(plans[-1:])
        own[d] = alone.launches() - 1
        alone.close()
    batch = mot.Batch(plans)
    launches = batch.launches() - 1
    batch.close()
    for p in plans:
        p.close()
    assert launches == sum(own[d] for d in lanes)
