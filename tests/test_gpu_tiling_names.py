"""The tiling that a context and a fit report is the one that runs: 0 names the
library's default rule, which no number of points stands for."""
import pytest

torch = pytest.importorskip("torch")

import paper_2104_14547_amd as nd  # noqa: E402
from tests.test_gpu_fit import T, make_fit, small_problem  # noqa: E402
from tests.test_gpu_tiles import batch_of  # noqa: E402
from tests.test_zz_no_alloc import uniform_inputs  # noqa: E402

pytestmark = pytest.mark.gpu


def test_context_reports_what_runs():
    b = batch_of(1, 3, 3, 12, 10, 700, 200, seed=1)
    (p, q, *_), x, g = uniform_inputs(b)
    run = lambda ctx: nd.api.surface_bwd(*x[:4], p, q, *x[4:], g, ctx=ctx)
    for set_to in (None, (0, 0), (0, 4096), (2048, 0), (16384, 16384)):
        a, c = nd.api.Context(0), nd.api.Context(0)
        if set_to:
            a.set_tiling(*set_to)
        assert a.tiling == (set_to or (0, 0))
        c.set_tiling(*a.tiling)
        assert all(torch.equal(u, v) for u, v in zip(run(a), run(c)))


def test_fit_reports_what_runs():
    s = small_problem(ns=200)
    make = lambda tiling: make_fit(s, graph=False, tiling=tiling)
    a = make(None)
    b = make(a.tiling)
    for f in (a, b):
        f.step(3)
    assert a.tiling == b.tiling == (0, 0)
    assert all(torch.equal(u, v) for u, v in zip(a.params, b.params))


def test_tuners_may_keep_the_default():
    assert 0 in nd.api.TILE_CANDIDATES and 0 in nd.fit.FIT_TILE_CANDIDATES
    b = batch_of(3, 2, 3, 14, 9, 300, 90, seed=2)
    args = [T(getattr(b, k)) for k in ("ctrl", "w", "ku", "kv", "us", "vs")]
    plan, report = nd.api.autotune(b.shapes, b.offsets, args, T(b.upstream), candidates=(0,), reps=2)
    assert report["chosen"]["fwd_tile_points"] == report["chosen"]["bwd_tile_points"] == 0
    for x, y in zip(plan.backward(*args, T(b.upstream)),
                    nd.SurfaceBatch(b.shapes, b.offsets).backward(*args, T(b.upstream))):
        assert torch.equal(x, y)
