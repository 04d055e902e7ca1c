"""How far a non-finite dL/dC of a curve reaches: the control points and knots
of its sample's own span and no others, whatever the samples' order, and an
infinity stays one where the sums hold no other."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_14547_amd as nd  # noqa: E402
from paper_2104_14547_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(torch.device("cuda", 0))


def spans_of(U, us, p):
    nc = len(U) - p - 1
    return np.clip(np.searchsorted(U, us, side="right") - 1, p, nc - 1)


@pytest.mark.parametrize("shuffle", [False, True])
@pytest.mark.parametrize("p,nc,ns,dim", [(3, 32, 1024, 3), (2, 9, 70, 2), (1, 60, 3000, 3), (5, 40, 385, 2)])
def test_nan_stays_with_its_span(p, nc, ns, dim, shuffle):
    cb = W.curve_batch(seed=p + ns, B=2, p=p, nc=nc, ns=ns, dim=dim, shared_u=False, shuffle=shuffle)
    args = [T(x) for x in (cb.ctrl, cb.w, cb.knots)]
    s = ns // 2
    k = int(spans_of(cb.knots[0], cb.us[0], p)[s])
    runs = {}
    for name, v in (("clean", cb.upstream[0, s, 0]), ("zero", 0.0), ("nan", np.nan)):
        g = cb.upstream.copy()
        g[0, s] = v if name != "clean" else g[0, s]
        runs[name] = [x.cpu().numpy() for x in nd.api.curve_bwd(*args, p, T(cb.us), T(g))]
    lo_hi = ((k - p, k + 1), (k - p, k + 1), (k - p + 1, k + p + 1))  # control points, weights, knots
    for clean, zero, nan, (lo, hi) in zip(runs["clean"], runs["zero"], runs["nan"], lo_hi):
        assert np.array_equal(nan[1], clean[1])
        out = np.ones(zero.shape[1], bool)
        out[lo:hi] = False
        assert np.isnan(nan[0][~out]).any()
        assert np.isfinite(nan[0][out]).all()
        # the sums of the other spans are the same terms, in another order at most
        assert np.abs(nan[0][out] - zero[0][out]).max(initial=0) <= 1e-4 * np.abs(zero[0]).max()


@pytest.mark.parametrize("shuffle", [False, True])
@pytest.mark.parametrize("p,nc,ns,dim", [(3, 12, 300, 3), (2, 5, 1000, 2), (1, 3, 2500, 3)])
def test_infinity_at_the_last_sample_of_every_span(p, nc, ns, dim, shuffle):
    cb = W.curve_batch(seed=ns, B=2, p=p, nc=nc, ns=ns, dim=dim, shared_u=False, shuffle=shuffle, repeat=0.0)
    cb.knots[:] = W.clamped_uniform_knots(nc, p)
    g = cb.upstream.copy()
    for c in range(2):
        k = spans_of(cb.knots[c], cb.us[c], p)
        for span in np.unique(k):
            at = np.flatnonzero(k == span)
            # the last in parameter for sorted samples, the last in input order otherwise
            g[c, at[-1], 0] = np.inf
    gc = nd.api.curve_bwd(*[T(x) for x in (cb.ctrl, cb.w, cb.knots)], p, T(cb.us), T(g))[0].cpu().numpy()
    # every basis function is positive strictly inside its spans
    assert np.isposinf(gc[..., 0]).all()
    assert np.isfinite(gc[..., 1:]).all()


def test_pairs_ordered_by_cell():
    # enough pairs to a cell that they are ordered: a NaN reaches its own cell
    p, q, nu_c, nv_c = 3, 2, 10, 9
    ub = W.uv_batch(seed=2, B=2, p=p, q=q, nu_c=nu_c, nv_c=nv_c, npts=40 * 7 * 7)
    args = [T(x) for x in (ub.ctrl, ub.w, ub.ku, ub.kv)]
    g = ub.upstream.copy()
    g[0, 100, 1] = np.nan
    clean, bad = ([x.cpu().numpy() for x in nd.api.surface_uv_bwd(*args, p, q, T(ub.uv), T(u))]
                  for u in (ub.upstream, g))
    ku, kv = (int(spans_of(U[0], ub.uv[0, 100:101, i], d)[0]) for i, (U, d) in enumerate(((ub.ku, p), (ub.kv, q))))
    own = np.zeros((nu_c, nv_c), bool)
    own[ku - p:ku + 1, kv - q:kv + 1] = True
    knots = []
    for n, k, d in ((nu_c + p + 1, ku, p), (nv_c + q + 1, kv, q)):
        own_k = np.zeros(n, bool)
        own_k[k - d + 1:k + d + 1] = True
        knots.append(own_k)
    for x, y, mine in zip(clean, bad, (own, own, *knots)):
        assert np.array_equal(x[1], y[1]) and np.array_equal(x[0][~mine], y[0][~mine])
        assert np.isnan(y[0][mine]).any()
