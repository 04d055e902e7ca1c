"""Workspace sizes: what the built-in scratch takes, and default tiles of narrow
grids."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_14547_amd as nd  # noqa: E402
from oracle import oracle as O  # noqa: E402
from tests.test_gpu_tiles import batch_of  # noqa: E402
from tests.test_zz_no_alloc import T, call_noalloc, uniform_inputs  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(3, 3, 48, 48, 2048, 2048), (3, 3, 128, 128, 1024, 1024), (3, 3, 48, 48, 100000, 4)])
def test_noalloc_takes_what_its_limit_admits(shape):
    # 22, 24 and 4 MiB counted in tiles of 16384 points
    b = batch_of(1, *shape, seed=sum(shape))
    dims, x, g = uniform_inputs(b)
    ctx = nd.api.Context(0)
    got = call_noalloc(ctx, dims, x, g)
    ref = nd.api.surface_bwd(*x[:4], dims[0], dims[1], *x[4:], g, ctx=ctx)
    for u, v in zip(got, ref):
        assert torch.equal(u, v)
    for t, ref in zip(got, O.bwd(b, b.upstream.astype(np.float64), local=True)):
        assert np.abs(t.cpu().numpy().ravel() - ref).max() <= 1e-4 * np.abs(ref).max()


@pytest.mark.parametrize("shape", [(3, 3, 16, 16, 100000, 1), (3, 2, 40, 60, 5000, 8), (2, 3, 9, 9, 300, 9)])
def test_narrow_grids_keep_their_slots_in_proportion(shape):
    p, q, nu_c, nv_c, nu_s, nv_s = shape
    b = batch_of(2, *shape, seed=sum(shape))
    sb = nd.SurfaceBatch(b.shapes, b.offsets)
    coarse = nd.api.Context(0)
    coarse.set_tiling(16384, 16384)
    most = max(nd.SurfaceBatch(b.shapes, b.offsets, ctx=coarse).ws_bytes, 2 * (16 * 12 * nu_s * nv_s + (1 << 20)))
    assert sb.ws_bytes <= nd.api.N.NURBS_PLAN_WS_HEADER + most
    packed = [T(getattr(b, k)) for k in ("ctrl", "w", "ku", "kv", "us", "vs")]
    got = sb.backward(*packed, T(b.upstream))
    dims, x, g = uniform_inputs(b)
    for u, v in zip(got, nd.api.surface_bwd(*x[:4], p, q, *x[4:], g)):
        assert torch.equal(u, v.ravel())
    for t, ref in zip(got, O.bwd(b, b.upstream.astype(np.float64), local=True)):
        for x, r in zip(t.cpu().numpy().reshape(2, -1), ref.reshape(2, -1)):
            assert np.abs(x - r).max() <= 1e-4 * np.abs(r).max()
