"""Gradients with the knots and parameters scaled by a power of two s and
dL/dS by another, t.  Both are exact, so dL/dP and dL/dw scale by t and dL/dU
by t / s, as long as no step forms a product out of the float range that the
result does not need: the square of a reciprocal knot interval, 2^136 or
2^-140 here, is such a one."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_14547_amd as nd  # noqa: E402
from paper_2104_14547_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu

SCALES = ((-62, -20), (76, 40))  # exponents of s and t


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(torch.device("cuda", 0))


def same(got, want, scales):
    for x, y, s in zip(got, want, scales):
        x, y = x.double() * 2.0 ** -s, y.double()
        # terms pushed below the normal range are a 2^-20 of the largest sums at most
        assert float((x - y).abs().max()) <= 2.0 ** -20 * float(y.abs().max())


@pytest.mark.parametrize("s,t", SCALES)
@pytest.mark.parametrize("p,dim", [(1, 2), (3, 3), (5, 2)])
def test_curve(p, dim, s, t):
    cb = W.curve_batch(seed=2, B=2, p=p, nc=60, ns=300, dim=dim, shared_u=False)
    cb.knots[:] = W.clamped_uniform_knots(60, p)
    run = lambda s, t: nd.api.curve_bwd(T(cb.ctrl), T(cb.w), T(cb.knots * 2.0 ** s), p, T(cb.us * 2.0 ** s),
                                        T(cb.upstream * 2.0 ** t))
    same(run(s, t), run(0, 0), (t, t, t - s))


@pytest.mark.parametrize("s,t", SCALES)
def test_grid_and_pairs(s, t):
    ub = W.uv_batch(seed=4, B=2, p=3, q=2, nu_c=50, nv_c=30, npts=3000)
    ku, kv = W.clamped_uniform_knots(50, 3), W.clamped_uniform_knots(30, 2)
    us, vs = W.uniform_grid(70), W.uniform_grid(66)
    up = np.random.Generator(np.random.PCG64(3)).uniform(-0.1, 0.1, (2, 70, 66, 3))

    def run(s, t):
        a, b = 2.0 ** s, 2.0 ** t
        net = (T(ub.ctrl), T(ub.w), T(np.stack([ku, ku]) * a), T(np.stack([kv, kv]) * a), 3, 2)
        return (nd.api.surface_bwd(*net, T(us * a), T(vs * a), T(up * b)),
                nd.api.surface_uv_bwd(*net, T(ub.uv * a), T(ub.upstream * b)))
    for got, want in zip(run(s, t), run(0, 0)):
        same(got, want, (t, t, t - s, t - s))
