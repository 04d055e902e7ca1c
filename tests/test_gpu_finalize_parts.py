"""dL/dP and dL/dw of uniform batches by the number of tiles of a surface (one,
two or three, more) and by the batch (a control point to a lane, or four where
the batch fills the chip all the same), at nets that fill no wave: within 1e-4
of the FP64 oracle, and the plan's gradients bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_14547_amd as nd  # noqa: E402
from oracle import oracle as O  # noqa: E402
from tests.test_gpu_tiles import batch_of  # noqa: E402
from tests.test_zz_no_alloc import T, uniform_inputs  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [2, 110])  # 150 waves of 64 control points a surface: 300, and over 16384
@pytest.mark.parametrize("nu_s,nv_s", [(40, 20), (150, 20), (60, 130), (200, 130)])  # 1, 2, 3 and 9 tiles
def test_parts(B, nu_s, nv_s):
    b = batch_of(B, 2, 3, 97, 99, nu_s, nv_s, seed=nu_s + nv_s)
    (p, q, *_), x, g = uniform_inputs(b)
    got = nd.api.surface_bwd(*x[:4], p, q, *x[4:], g)
    packed = [T(getattr(b, k)) for k in ("ctrl", "w", "ku", "kv", "us", "vs")]
    for u, v in zip(got, nd.SurfaceBatch(b.shapes, b.offsets).backward(*packed, T(b.upstream))):
        assert torch.equal(u.ravel(), v)
    for t, ref in zip(got, O.bwd(b, b.upstream.astype(np.float64), local=True)):
        t, ref = t.cpu().numpy().reshape(B, -1), ref.reshape(B, -1)
        assert (np.abs(t - ref).max(1) <= 1e-4 * np.abs(ref).max(1)).all()
