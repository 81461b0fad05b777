"""The binning sort at the sizes where its launches change, against the oracle's counting sort."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("npts", [1, 1024, 1025, 2049, 4097, 8193, 40000])  # one block; one, two, three strides ...
def test_bin_points_of_every_pass_count(npts):
    from paper_2208_03120_amd import mot
    r = np.random.Generator(np.random.PCG64(npts))
    x = r.uniform(-0.3, 0.3, size=(npts, 2))
    s, o = np.full(2, 32.0), np.full(2, 32.0)
    cell, perm, toff = mot.bin_points(x, s, o, 64, 8)
    ocell, _, operm, otoff = oracle.bin_points(x, s, o, 64, 8)
    np.testing.assert_array_equal(cell, ocell)
    np.testing.assert_array_equal(perm, operm)
    np.testing.assert_array_equal(toff, otoff)
