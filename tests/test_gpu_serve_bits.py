"""A served result has the bits of a uniform call with tiles of 16384 points."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_14547_amd as nd  # noqa: E402
from paper_2104_14547_amd import workloads as W  # noqa: E402
from paper_2104_14547_amd.serve import Server, make_requests, run_load  # noqa: E402

pytestmark = pytest.mark.gpu


def test_bits_of_a_call_with_16384_points_to_a_tile():
    pool = W.uneven_batch(3, n_surf=24, with_upstream=False)
    reqs = make_requests(pool, 24, seed=5)
    with Server(pool, slot_bytes=256 << 20, n_slots=2, max_requests=16) as srv:
        _, res = run_load(srv, reqs, rate=None)
    ctx = nd.api.Context(0)
    ctx.set_tiling(16384, 16384)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    for (s, us, vs, target), r in zip(reqs, res):
        d = pool.surface(s)
        args = (T(d["ctrl"]), T(d["w"]), T(d["ku"]), T(d["kv"]), d["p"], d["q"], T(us), T(vs))
        pts = nd.api.surface_fwd(*args, ctx=ctx)
        grads = nd.api.surface_bwd(*args, 2.0 * (pts - T(target)), ctx=ctx)
        for x, y in zip((pts, *grads), (r.pts, r.grad_ctrl, r.grad_w, r.grad_ku, r.grad_kv)):
            assert np.array_equal(x.cpu().numpy().ravel(), y.ravel())
