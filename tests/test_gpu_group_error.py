"""Rounding of products that share their points (grouped spreading and interpolation): scaling
vectors of row-by-row circles after three sweeps against the same iterations in FP64.

Job by job the kernels give 3.8e-8 with the scalings rounded to FP32 (2.4e-8 of it), one FP32 chain
for a quarter of a result's terms gave 5.4e-8; without that rounding 2.9e-8 and 4.8e-8.  The
bound lies half way."""
import numpy as np
import pytest

from paper_2208_03120_amd import workloads as W

pytestmark = pytest.mark.gpu


def exact_circle(X, mu, eta, sweeps):
    K = len(X)

    def kmat(a, b):
        return np.exp(-((a[:, None] - b[None]) ** 2).sum(-1) / eta)

    edge = [kmat(X[k], X[k + 1]) for k in range(K - 1)]
    phi = [np.ones(len(x)) for x in X]
    beta = [None] * K
    beta[K - 1] = kmat(X[0], X[K - 1])

    def up():
        for k in range(K - 2, 0, -1):
            beta[k] = (beta[k + 1] * phi[k + 1]) @ edge[k].T

    up()
    for _ in range(sweeps):
        phi[0] = mu[0] / ((edge[0] * beta[1]) @ phi[1])
        g = edge[0]
        for k in range(1, K):
            if k > 1:
                g = (g * phi[k - 1]) @ edge[k - 1]
            phi[k] = mu[k] / (phi[0] @ (beta[k] * g))
        up()
    return np.concatenate(phi)


@pytest.mark.parametrize("seed", [0, 1])
def test_circle_2d(seed):
    from paper_2208_03120_amd import mot
    inst = W.make_instance(np.random.Generator(np.random.PCG64(seed)), 4, 1500, 2, W.CIRCLE, 0.2)
    plan = mot.Plan(inst.points, inst.weights, W.CIRCLE, None, inst.eta, path=mot.NFFT)
    plan.sinkhorn(3)
    got = np.concatenate(plan.scalings())
    plan.close()
    want = exact_circle(inst.points, inst.weights, inst.eta, 3)
    assert np.linalg.norm(got - want) < 3.8e-8 * np.linalg.norm(want)


@pytest.mark.parametrize("d,rows", [(2, 511), (2, 512), (2, 545), (1, 1279), (1, 1280), (1, 1345)])
def test_rows_around_the_grouping(d, rows):
    """Circles of as many rows as are still spread and interpolated job by job, the fewest that are
    grouped, and a number that leaves a last group of one; marginals down to one point."""
    import oracle
    from paper_2208_03120_amd import mot
    inst = W.make_instance(np.random.Generator(np.random.PCG64(rows)), 4, [rows, 130, 17, 1], d, W.CIRCLE, 0.1)
    plan = mot.Plan(inst.points, inst.weights, W.CIRCLE, None, inst.eta, path=mot.NFFT)
    plan.sinkhorn(2)
    got = plan.scalings()
    plan.close()
    want = oracle.circle_sinkhorn(inst.points, inst.weights, inst.eta, 2)[0]
    for a, b in zip(got, want):
        np.testing.assert_allclose(a, b, rtol=1e-5)
