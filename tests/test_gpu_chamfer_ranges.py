"""Nearest points over 1 to 33 ranges of 64 targets, which are compared sixteen
and eight at a time: indices and d2 bit for bit as the oracle's ordered scan."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_14547_amd as nd  # noqa: E402
from paper_2104_14547_amd import workloads as W  # noqa: E402
from oracle import oracle as O  # noqa: E402
from tests.test_gpu_chamfer import H, T, check_pair  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ranges", [1, 7, 8, 9, 15, 16, 17, 24, 25, 32, 33])
def test_ranges(ranges):
    for lattice in (False, True):
        P, Q = W.point_sets(seed=ranges, B=2, n=5, m=64 * ranges - 3, dim=3, lattice=lattice)
        idx, d2 = nd.api.nearest(T(P), T(Q))
        out = nd.api.chamfer_hausdorff(T(P), T(Q))
        for b in range(2):
            ri, rd = O.nearest(P[b], Q[b])
            np.testing.assert_array_equal(H(idx[b]), ri)
            np.testing.assert_array_equal(H(d2[b]), rd)
            check_pair(P[b], Q[b], *[x[b] for x in out])
