"""Nearest points at the edges of their search: target groups of 16, ranges of
64 and 256, 256 queries to a workgroup, one, two and four queries to a lane, a
group with several targets at the least distance, and distances that are not
numbers.  Indices and d2 bit for bit as the oracle's ordered scan."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_14547_amd as nd  # noqa: E402
from paper_2104_14547_amd import workloads as W  # noqa: E402
from oracle import oracle as O  # noqa: E402
from tests.test_gpu_chamfer import H, T, check_pair  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,n,m", [(1, 256, 15), (1, 257, 16), (2, 5, 17), (1, 1024, 63), (1, 1025, 65), (3, 255, 257),
                                   (1, 40000, 300), (300, 30, 100), (1, 300, 20000)])
def test_search_edges(B, n, m):
    for lattice in (False, True):
        P, Q = W.point_sets(seed=n + 7 * m, B=B, n=n, m=m, dim=3, lattice=lattice)
        idx, d2 = nd.api.nearest(T(P), T(Q))
        cd, hd, gcd, ghd = nd.api.chamfer_hausdorff(T(P), T(Q))
        for b in sorted({0, B // 2, B - 1}):
            ri, rd = O.nearest(P[b], Q[b])
            np.testing.assert_array_equal(H(idx[b]), ri)
            np.testing.assert_array_equal(H(d2[b]), rd)
            check_pair(P[b], Q[b], cd[b], hd[b], gcd[b], ghd[b])


def test_not_a_number_and_infinity():
    P, Q = W.point_sets(seed=3, B=1, n=400, m=900, dim=3)
    Q[0, 17] = np.nan
    Q[0, 600:] = np.inf
    P[0, 5] = np.nan
    idx, d2 = (H(t) for t in nd.api.nearest(T(P[0]), T(Q[0])))
    keep = np.isfinite(Q[0]).all(1)
    ri, rd = O.nearest(np.delete(P[0], 5, 0), Q[0][keep])
    np.testing.assert_array_equal(np.delete(idx, 5), np.flatnonzero(keep)[ri])
    np.testing.assert_array_equal(np.delete(d2, 5), rd)
    assert idx[5] == 0 and np.isnan(d2[5])
    # no distance is a number: the call ends, with indices in range
    cd, hd, gcd, ghd = nd.api.chamfer_hausdorff(T(np.full_like(P[0], np.nan)), T(Q[0]))
    assert np.isnan(float(cd)) and gcd.shape == (400, 3)
