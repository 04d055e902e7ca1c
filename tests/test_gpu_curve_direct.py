"""Curves where their split changes: samples taken as they come (at most four to
a span, sorted) or in items, one, two or four waves, as many spans in use as a
workgroup has lanes, so that items have to be shared out, and the forward with
and without its table; sorted and unsorted.  Bars as for the other curve tests,
and the same bits in any batch."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_14547_amd as nd  # noqa: E402
from paper_2104_14547_amd import workloads as W  # noqa: E402
from tests.test_gpu_curves import T, run_case  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shuffle", [False, True])
@pytest.mark.parametrize("p,nc,ns,dim", [
    (3, 67, 64, 3), (3, 67, 65, 2), (3, 67, 128, 3), (3, 67, 129, 3), (3, 67, 256, 3), (3, 67, 257, 3), (5, 69, 256, 2),
    (1, 64, 300, 2), (2, 66, 384, 3), (3, 240, 1024, 3), (1, 240, 1912, 2), (1, 240, 1913, 2), (7, 200, 2500, 3),
    (2, 9, 511, 2), (2, 9, 512, 3), (4, 30, 255, 2), (4, 30, 256, 3)])
def test_split(p, nc, ns, dim, shuffle):
    cb = W.curve_batch(seed=p * ns + nc, B=3, p=p, nc=nc, ns=ns, dim=dim, shared_u=False, shuffle=shuffle, repeat=0.1)
    run_case(cb, derivs=False)
    args = [T(x) for x in (cb.ctrl, cb.w, cb.knots, cb.us, cb.upstream)]
    many = nd.api.curve_bwd(*args[:3], p, *args[3:])
    one = nd.api.curve_bwd(*[x[1:2] for x in args[:3]], p, *[x[1:2] for x in args[3:]])
    assert all(torch.equal(x[1:2], y) for x, y in zip(many, one))


def test_spans_of_unequal_numbers_of_samples():
    # half the samples in one of 63 spans
    cb = W.curve_batch(seed=9, B=2, p=2, nc=65, ns=380, dim=3, shared_u=False)
    cb.knots[:] = W.clamped_uniform_knots(65, 2)
    cb.us[:, 100:290] = np.linspace(cb.knots[0, 30], cb.knots[0, 31], 190, endpoint=False, dtype=np.float32)
    cb.us.sort(axis=1)
    run_case(cb, derivs=False)
