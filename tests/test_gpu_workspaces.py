"""Workspace sizes: what the built-in scratch takes, default tiles of narrow
grids, and a workspace sized for a larger call serving a smaller one."""
import ctypes
import random

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_14547_amd as nd  # noqa: E402
from paper_2104_14547_amd import _native as N  # noqa: E402
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


@pytest.mark.parametrize("shape", [(3, 3, 16, 16, 100000, 1), (3, 2, 40, 60, 5000, 4), (2, 3, 9, 9, 300, 5)])
def test_narrow_grids_keep_their_slots_in_proportion(shape):
    p, q, nu_c, nv_c, nu_s, nv_s = shape
    b = batch_of(2, *shape, seed=sum(shape))
    sb = nd.SurfaceBatch(b.shapes, b.offsets)
    coarse = nd.api.Context(0)
    coarse.set_tiling(16384, 16384)
    most = max(nd.SurfaceBatch(b.shapes, b.offsets, ctx=coarse).ws_bytes, 2 * (16 * 12 * nu_s * nv_s + (1 << 20)))
    assert sb.ws_bytes <= N.NURBS_PLAN_WS_HEADER + most
    packed = [T(getattr(b, k)) for k in ("ctrl", "w", "ku", "kv", "us", "vs")]
    got = sb.backward(*packed, T(b.upstream))
    dims, x, g = uniform_inputs(b)
    for u, v in zip(got, nd.api.surface_bwd(*x[:4], p, q, *x[4:], g)):
        assert torch.equal(u, v.ravel())
    for t, ref in zip(got, O.bwd(b, b.upstream.astype(np.float64), local=True)):
        for x, r in zip(t.cpu().numpy().reshape(2, -1), ref.reshape(2, -1)):
            assert np.abs(x - r).max() <= 1e-4 * np.abs(r).max()


def asked(ctx, shape, B):
    p, q, nu_c, nv_c, nu_s, nv_s = shape
    n = ctypes.c_size_t()
    assert N.lib().nurbs_surface_ws_bytes(ctx.handle, B, p, q, nu_c, nv_c, nu_s, nv_s, 15, ctypes.byref(n)) == 0
    return n.value


def needed(ctx, shape, B):
    """What the call itself requires, from its refusal of one byte (no pointer is followed)."""
    p, q, nu_c, nv_c, nu_s, nv_s = shape
    rc = N.lib().nurbs_surface_bwd(ctx.handle, B, p, q, nu_c, nv_c, 256, 256, 256, 256, nu_s, nv_s, 256, 256, 1, 256,
                                   256, 256, 256, 256, 15, 256, 1, None)
    assert rc == N.NURBS_EWORKSPACE
    return int(N.lib().nurbs_last_error(ctx.handle).decode().split("need ")[1])


def test_asked_workspace_grows_with_every_size():
    rnd = random.Random(7)
    ctx = nd.api.Context(0)
    for _ in range(3000):
        p, q = rnd.randint(1, 7), rnd.randint(1, 7)
        big = [p, q, rnd.randint(p + 1, 200), rnd.randint(q + 1, 200), int(2 ** rnd.uniform(0, 17)),
               int(2 ** rnd.uniform(0, 10))]
        small = [rnd.randint(1, p), rnd.randint(1, q)]
        for d, b in zip(small, big[2:4]):
            small.append(rnd.randint(d + 1, b))
        for b in big[4:]:
            small.append(rnd.choice([b, max(1, b - 1), rnd.randint(1, b)]))
        if rnd.random() < 0.5:
            small[:4] = big[:4]
        B = rnd.choice([1, 3, 40, 1000])
        b = rnd.choice([B, rnd.randint(1, B)])
        assert needed(ctx, small, b) <= asked(ctx, small, b) <= asked(ctx, big, B), (big, B, small, b)


@pytest.mark.parametrize("tab", [False, True])
def test_workspace_of_a_larger_call_serves_a_smaller_one(tab):
    # tiles of one row: 148 and 134 MB of slots a surface, so that a gibibyte
    # holds seven of the larger and eight of the smaller
    ctx = nd.api.Context(0)
    ctx.set_tiling(64, 64)
    big, small = (3, 3, 64, 64, 1085, 64), (3, 3, 64, 64, 980, 64)
    n = asked(ctx, big, 8)
    assert needed(ctx, small, 8) <= n
    b = batch_of(8, *small, seed=3)
    (p, q, *sizes), (ctrl, w, ku, kv, us, vs), g = uniform_inputs(b)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    got = [torch.full_like(t, float("nan")) for t in (ctrl, w)]
    at = [t.data_ptr() for t in (ctrl, w, ku, kv)]
    if tab:
        nu, nv = nd.api.basis_table(ku, p, us), nd.api.basis_table(kv, q, vs)
        rc = N.lib().nurbs_surface_bwd_tab(
            ctx.handle, 8, p, q, 64, 64, *at, 980, 64, us.data_ptr(), vs.data_ptr(), 0, nu.data_ptr(), nv.data_ptr(), 0,
            g.data_ptr(), got[0].data_ptr(), got[1].data_ptr(), 3, ws.data_ptr(), n, nd.api._stream(ctrl.device))
    else:
        rc = N.lib().nurbs_surface_bwd(
            ctx.handle, 8, p, q, 64, 64, *at, 980, 64, us.data_ptr(), vs.data_ptr(), 0, g.data_ptr(),
            got[0].data_ptr(), got[1].data_ptr(), None, None, 3, ws.data_ptr(), n, nd.api._stream(ctrl.device))
    assert rc == 0, N.lib().nurbs_last_error(ctx.handle).decode()
    # a group of seven and one of one: the bits of each surface alone
    for i in (0, 6, 7):
        args = (ctrl[i], w[i], ku[i], kv[i], p, q, us[i], vs[i])
        if tab:
            ref = nd.api.surface_bwd_tab(*args, nu[i:i + 1], nv[i:i + 1], g[i], ctx=ctx)
        else:
            ref = nd.api.surface_bwd(*args, g[i], mask=3, ctx=ctx)
        assert torch.equal(got[0][i], ref[0]) and torch.equal(got[1][i], ref[1])
    for t, ref in zip(got, O.bwd(b, b.upstream.astype(np.float64), local=True)):
        for x, r in zip(t.cpu().numpy().reshape(8, -1), ref.reshape(8, -1)):
            assert np.abs(x - r).max() <= 1e-4 * np.abs(r).max()
