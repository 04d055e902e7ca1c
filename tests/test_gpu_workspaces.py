"""Workspace sizes: what the built-in scratch takes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_14547_amd as nd  # noqa: E402
from oracle import oracle as O  # noqa: E402
from tests.test_gpu_tiles import batch_of  # noqa: E402
from tests.test_zz_no_alloc import call_noalloc, uniform_inputs  # noqa: E402

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
