"""Scattered backward over pairs ordered by cell, at the sizes where it can go
wrong: one pair, a wave's remainder, a cell cut into items (one cell holds all
pairs of a Bezier net), the longer items of large inputs, the most cells the
ordering counts in LDS and one row more (the atomic path), a pair fewer than
cells (the atomic path), every degree class, and
a workspace too small for the tables (the atomic path).

Bars as for the other scattered tests: each gradient within 1e-4 of its
tensor's largest magnitude in the FP64 oracle, per surface.
"""
import ctypes

import pytest

torch = pytest.importorskip("torch")

import paper_2104_14547_amd as nd  # noqa: E402
from paper_2104_14547_amd import workloads as W  # noqa: E402
from tests.test_gpu_uv import T, run_case  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,q,nu_c,nv_c,npts,B", [
    (3, 3, 4, 4, 1, 2), (3, 2, 4, 3, 129, 2), (2, 2, 3, 3, 33000, 1), (7, 7, 9, 8, 513, 2), (5, 2, 6, 30, 4000, 1),
    (1, 1, 65, 65, 5000, 1), (1, 1, 66, 65, 5000, 1), (6, 4, 20, 31, 3001, 2), (2, 3, 10, 10, 56, 2), (2, 3, 10, 10, 55, 2)])
def test_cells_parity(p, q, nu_c, nv_c, npts, B):
    ub = W.uv_batch(seed=31 + npts, B=B, p=p, q=q, nu_c=nu_c, nv_c=nv_c, npts=npts, repeat=0.15)
    _, a = run_case(ub, derivs=False)
    args = [T(x) for x in (ub.ctrl, ub.w, ub.ku, ub.kv)]
    # bitwise: again, each surface alone, and each gradient alone
    b = nd.api.surface_uv_bwd(*args, p, q, T(ub.uv), T(ub.upstream))
    assert all(torch.equal(x, y) for x, y in zip(a, b))
    one = nd.api.surface_uv_bwd(*[x[B - 1] for x in args], p, q, T(ub.uv[B - 1]), T(ub.upstream[B - 1]))
    assert all(torch.equal(x[B - 1], y) for x, y in zip(a, one))
    for i in range(4):
        c = nd.api.surface_uv_bwd(*args, p, q, T(ub.uv), T(ub.upstream), mask=1 << i)
        assert torch.equal(c[i], a[i]) and all(c[j] is None for j in range(4) if j != i)


def test_small_workspace_takes_the_atomic_path():
    N = nd.api.N
    ub = W.uv_batch(seed=8, B=2, p=3, q=3, nu_c=10, nv_c=11, npts=3000)
    ctx = nd.api.context(0)
    sizes = []
    for npts in (0, ub.npts):
        n = ctypes.c_size_t()
        nd.api._check(N.lib().nurbs_surface_uv_ws_bytes(ctx.handle, 2, 3, 3, 10, 11, npts, 15, ctypes.byref(n)))
        sizes.append(n.value)
    assert sizes[0] < sizes[1]
    _, want = run_case(ub, derivs=False)
    ten = [T(x) for x in (ub.ctrl, ub.w, ub.ku, ub.kv, ub.uv, ub.upstream)]
    got = [torch.empty_like(x) for x in ten[:4]]
    ws = torch.empty(sizes[0], dtype=torch.uint8, device="cuda")
    ptr = [x.data_ptr() for x in ten]
    nd.api._check(N.lib().nurbs_surface_uv_bwd(
        ctx.handle, 2, 3, 3, 10, 11, *ptr[:4], ub.npts, ptr[4], 0, ptr[5], *[x.data_ptr() for x in got], 15,
        ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream))
    # both paths are within 1e-4 of the oracle, so within 2e-4 of each other
    for x, y in zip(got, want):
        assert float((x - y).abs().max()) <= 2e-4 * float(y.abs().max())
