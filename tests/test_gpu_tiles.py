"""Grid tiles at the sizes where their split can go wrong: one to over 64
tiles per surface (the finalize looks at 64 headers at a time), one to many
64-sample chunks of a knot vector shared by a workgroup's waves, sample counts
at the edge where they start to share, and a batch taken in groups.

Gradients within 1e-4 of each tensor's largest magnitude in the FP64 oracle,
points equal bit for bit for every forward tiling, and the uniform call equal
to the plan bit for bit under one backward tiling.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_14547_amd as nd  # noqa: E402
from paper_2104_14547_amd import workloads as W  # noqa: E402
from tests.test_gpu_parity import H, T, check_grads, check_points, oracle_both  # noqa: E402
from tests.test_zz_no_alloc import call_noalloc, check_against_oracle, uniform_inputs, with_upstream  # noqa: E402

pytestmark = pytest.mark.gpu


def batch_of(B, p, q, nu_c, nv_c, nu_s, nv_s, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    parts = [dict(p=p, q=q, nu_c=nu_c, nv_c=nv_c, nu_s=nu_s, nv_s=nv_s, ctrl=W.perturbed_lattice(g, nu_c, nv_c),
                  w=g.uniform(0.5, 1.5, (nu_c, nv_c)), ku=W.clamped_random_knots(g, nu_c, p, 0.2),
                  kv=W.clamped_random_knots(g, nv_c, q, 0.2), us=W.uniform_grid(nu_s), vs=W.uniform_grid(nv_s))
             for _ in range(B)]
    return with_upstream(W.pack("tiles", parts), seed + 1)


@pytest.mark.parametrize("shape,tile", [
    ((3, 2, 40, 9, 1030, 70), 256), ((2, 3, 12, 30, 64, 64), 0), ((2, 3, 12, 30, 65, 64), 0),
    ((4, 1, 9, 40, 64, 65), 512), ((3, 3, 70, 66, 300, 300), 64), ((1, 5, 2, 6, 1, 600), 0),
    ((7, 7, 9, 9, 257, 3), 1024)])
def test_tiles(shape, tile):
    p, q, nu_c, nv_c, nu_s, nv_s = shape
    b = batch_of(2, *shape, seed=sum(shape))
    S, G = oracle_both(b, b.upstream)
    sh, x, g = uniform_inputs(b)
    ctx = nd.api.Context(0)
    ctx.set_tiling(tile, tile)
    args = (*x[:4], p, q, *x[4:])
    pts = nd.api.surface_fwd(*args, ctx=ctx)
    check_points(b, H(pts).ravel(), S)
    for t in (0, 64, 1024, 16384):
        other = nd.api.Context(0)
        other.set_tiling(t, t)
        assert torch.equal(nd.api.surface_fwd(*args, ctx=other), pts)
    grads = nd.api.surface_bwd(*args, g, ctx=ctx)
    check_grads(b, [H(t).ravel() for t in grads], G)
    sb = nd.SurfaceBatch(b.shapes, b.offsets, ctx=ctx)
    packed = [T(getattr(b, k)) for k in ("ctrl", "w", "ku", "kv", "us", "vs")]
    assert torch.equal(sb.forward(*packed), pts.ravel())
    for u, v in zip(sb.backward(*packed, T(b.upstream)), grads):
        assert torch.equal(u, v.ravel())


def test_groups_give_the_same_bits():
    # 30 surfaces of seven tiles with 2.4 MB of slots: two groups in the
    # built-in scratch, one in a workspace
    b = batch_of(30, 2, 3, 250, 20, 512, 64, seed=5)
    shape, x, g = uniform_inputs(b)
    ctx = nd.api.Context(0)
    got = call_noalloc(ctx, shape, x, g)
    ref = nd.api.surface_bwd(*x[:4], shape[0], shape[1], *x[4:], g, ctx=ctx)
    for u, v in zip(got, ref):
        assert torch.equal(u, v)
    check_against_oracle(b, got)
