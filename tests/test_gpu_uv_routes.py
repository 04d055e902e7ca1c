"""Scattered backward on both sides of the line between its two paths, the
degrees of the atomic one, its workspaces and its groups of surfaces.

Bars as for the other scattered tests: each gradient within 1e-4 of its
tensor's largest magnitude in the FP64 oracle, per surface.
"""
import ctypes
import random

import pytest

torch = pytest.importorskip("torch")

import paper_2104_14547_amd as nd  # noqa: E402
from paper_2104_14547_amd import workloads as W  # noqa: E402
from tests.test_gpu_uv import T, run_case  # noqa: E402

pytestmark = pytest.mark.gpu
N = nd.api.N


def check(p, q, nu_c, nv_c, npts, B):
    ub = W.uv_batch(seed=17 + npts, B=B, p=p, q=q, nu_c=nu_c, nv_c=nv_c, npts=npts, repeat=0.15)
    _, a = run_case(ub, derivs=False)
    # bitwise: each surface alone
    one = nd.api.surface_uv_bwd(*[T(x[B - 1]) for x in (ub.ctrl, ub.w, ub.ku, ub.kv)], p, q, T(ub.uv[B - 1]),
                                T(ub.upstream[B - 1]))
    assert all(torch.equal(x[B - 1], y) for x, y in zip(a, one))


# few pairs to a cell, accumulators in LDS (20 x 18) and in global memory (48 x 44)
@pytest.mark.parametrize("p,q", [(1, 1), (2, 3), (4, 4), (5, 5), (6, 2), (4, 7), (7, 7)])
@pytest.mark.parametrize("nu_c,nv_c,npts", [(20, 18, 500), (48, 44, 900)])
def test_few_pairs_to_a_cell(p, q, nu_c, nv_c, npts):
    check(p, q, nu_c, nv_c, npts, 2)


@pytest.mark.parametrize("p,q,nu_c,nv_c,least", [
    (3, 3, 9, 8, 32), (1, 1, 9, 7, 96), (7, 6, 12, 9, 32), (2, 4, 40, 41, 32), (1, 1, 65, 65, 2), (5, 4, 44, 43, 1),
    (1, 2, 44, 43, 1)])
def test_both_sides_of_the_line(p, q, nu_c, nv_c, least):
    line = least * (nu_c - p) * (nv_c - q)
    for npts in (line - 1, line):
        check(p, q, nu_c, nv_c, npts, 2)



def asked(B, p, q, nu_c, nv_c, npts):
    n = ctypes.c_size_t()
    assert N.lib().nurbs_surface_uv_ws_bytes(nd.api.context(0).handle, B, p, q, nu_c, nv_c, npts, 15, ctypes.byref(n)) == 0
    return n.value


def test_asked_workspace_grows_with_every_size():
    rnd = random.Random(5)
    for _ in range(3000):
        p, q = rnd.randint(1, 7), rnd.randint(1, 7)
        big = [p, q, rnd.randint(p + 1, 100), rnd.randint(q + 1, 100), int(2 ** rnd.uniform(0, 21))]
        small = [rnd.randint(1, p), rnd.randint(1, q)]
        small += [rnd.choice([b, rnd.randint(d + 1, b)]) for d, b in zip(small, big[2:])]
        small.append(rnd.choice([big[4], max(1, big[4] - 1), rnd.randint(1, big[4])]))
        B = rnd.choice([1, 3, 40, 2000])
        assert asked(rnd.randint(1, B), *small) <= asked(B, *big), (B, big, small)


@pytest.mark.parametrize("big,small", [
    ((1, 3, 3, 20, 20, 32768), (1, 3, 3, 20, 20, 32767)),  # shorter items
    ((2, 1, 1, 60, 60, 16385), (2, 1, 1, 60, 60, 16384)),  # more chunks
    ((1, 7, 7, 48, 46, 9000), (1, 1, 1, 48, 46, 9000)),    # more cells
    ((3, 3, 3, 20, 20, 300), (1, 3, 3, 4, 4, 300))])       # the larger call takes the atomic path
def test_workspace_of_a_larger_call_serves_a_smaller_one(big, small):
    B, p, q, nu_c, nv_c, npts = small
    ub = W.uv_batch(seed=npts, B=B, p=p, q=q, nu_c=nu_c, nv_c=nv_c, npts=npts)
    _, want = run_case(ub, derivs=False)
    ten = [T(x) for x in (ub.ctrl, ub.w, ub.ku, ub.kv, ub.uv, ub.upstream)]
    got = [torch.full_like(x, float("nan")) for x in ten[:4]]
    ws = torch.empty(asked(*big), dtype=torch.uint8, device="cuda")
    ptr = [x.data_ptr() for x in ten]
    ctx = nd.api.context(0)
    nd.api._check(N.lib().nurbs_surface_uv_bwd(
        ctx.handle, B, p, q, nu_c, nv_c, *ptr[:4], npts, ptr[4], 0, ptr[5], *[x.data_ptr() for x in got], 15,
        ws.data_ptr(), ws.numel(), nd.api._stream(ws.device)), ctx.handle)
    assert all(torch.equal(x, y) for x, y in zip(got, want))


def test_batch_in_groups():
    # 2.5 MB of tables and slots a surface: two groups in a gibibyte
    B, p, q, nc, npts = 450, 5, 5, 48, 2000
    ub = W.uv_batch(seed=1, B=9, p=p, q=q, nu_c=nc, nv_c=nc, npts=npts)
    args = [T(x) for x in (ub.ctrl, ub.w, ub.ku, ub.kv, ub.uv, ub.upstream)]
    assert asked(B, p, q, nc, nc, npts) < 50 * asked(9, p, q, nc, nc, npts)
    many = [x.repeat(50, *[1] * (x.dim() - 1)) for x in args]
    got = nd.api.surface_uv_bwd(*many[:4], p, q, *many[4:])
    _, want = run_case(ub, derivs=False)
    for x, y in zip(got, want):
        assert torch.equal(x.reshape(50, 9, -1), y.reshape(1, 9, -1).expand(50, -1, -1))
