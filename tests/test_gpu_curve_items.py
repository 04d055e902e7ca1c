"""Curve backward at the sizes where its span order and items can go wrong:
one sample, a lane's and a wave's remainder, one span holding all samples,
more spans than samples, every parameter equal, a full chunk and one sample
more, the longest polygon at the largest degree; sorted and unsorted, in the
plane and in space.  Bars as for the other curve tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_14547_amd as nd  # noqa: E402
from paper_2104_14547_amd import workloads as W  # noqa: E402
from tests.test_gpu_curves import T, run_case  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shuffle", [False, True])
@pytest.mark.parametrize("p,nc,ns,dim", [(3, 4, 1, 3), (2, 3, 9, 2), (1, 2, 2048, 3), (3, 40, 17, 3), (5, 23, 513, 2),
                                         (4, 9, 2049, 3), (7, 248, 2000, 3), (7, 8, 64, 2)])
def test_curve_items_parity(p, nc, ns, dim, shuffle):
    cb = W.curve_batch(seed=p * ns + nc, B=2, p=p, nc=nc, ns=ns, dim=dim, shared_u=False, shuffle=shuffle, repeat=0.15)
    run_case(cb, derivs=False)


@pytest.mark.parametrize("spans", [63, 64, 65, 128])
def test_as_many_spans_as_lanes(spans):
    # every span holds samples, one item each at least: the item length has to
    # exist where spans and lanes are equal in number
    cb = W.curve_batch(seed=spans, B=2, p=1, nc=spans + 1, ns=300, dim=2)
    cb.knots[:] = W.clamped_uniform_knots(spans + 1, 1)
    run_case(cb, derivs=False)


def test_one_parameter_for_all_samples_and_order_invariance():
    cb = W.curve_batch(seed=1, B=2, p=3, nc=12, ns=300, dim=3, shared_u=False)
    cb.us[0] = cb.us[0, 150]
    run_case(cb, derivs=False)
    # descending parameters take the sort; the gradients do not depend on the
    # order beyond the rounding of their sums (300 terms of one sign at most)
    args = [T(x) for x in (cb.ctrl, cb.w, cb.knots)]
    a = nd.api.curve_bwd(*args, 3, T(cb.us), T(cb.upstream))
    b = nd.api.curve_bwd(*args, 3, T(cb.us[:, ::-1]), T(cb.upstream[:, ::-1]))
    for x, y in zip(a, b):
        assert float((x - y).abs().max()) <= 1e-4 * float(x.abs().max())
