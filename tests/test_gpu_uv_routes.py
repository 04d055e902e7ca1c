"""Scattered backward on both sides of the line between its two paths, and the
degrees of the atomic one.

Bars as for the other scattered tests: each gradient within 1e-4 of its
tensor's largest magnitude in the FP64 oracle, per surface.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_14547_amd as nd  # noqa: E402
from paper_2104_14547_amd import workloads as W  # noqa: E402
from tests.test_gpu_uv import T, run_case  # noqa: E402

pytestmark = pytest.mark.gpu


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

