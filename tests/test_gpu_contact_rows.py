"""The contact search's rows of grid cells: pairs of 12-vertex cells at many places of the
grid, so that rows start at every part of the (1024-entry) hash table, some of them running
over its end, against all pairs of vertices.  Positions are sums of two doubles on both
sides; the partner is exact where no second candidate is within rounding of the nearest."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from rbc_inputs import meshes
from test_gpu_parity import T, make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_contacts_in_rows_over_the_whole_table(precision):
    from paper_1903_06479_amd import Batch
    X, Tr = meshes.sphere_mesh(12, 1.0)
    n = len(X)
    plan = make([(X, Tr)], precision)
    batch = Batch(plan, np.zeros(2, np.int32))
    rng = np.random.default_rng(5)
    x = np.concatenate([X, X @ np.linalg.qr(rng.standard_normal((3, 3)))[0]]).astype(np.float32).astype(np.float64)
    found = 0
    for _ in range(150):
        origin = rng.uniform(-900.0, 900.0, 3) + np.array([[0.0, 0.0, 0.0], [0.3, 1.1, -0.4]])
        q, nn, count = batch.detect_contacts(T(origin, torch.float64), T(x, plan.torch_dtype), 1.0, count=True)
        q, nn = q.cpu().numpy().astype(np.float64), nn.cpu().numpy()
        w = (origin[:, None] + x.reshape(2, n, 3))
        d = np.linalg.norm(w[0][:, None] - w[1][None], axis=2)
        for c, dist in ((0, d), (1, d.T)):
            j = dist.argmin(1)
            near = dist[np.arange(n), j]
            has = np.any(nn[c * n:(c + 1) * n] != 0, axis=1)
            sure = np.abs(near - 1.0) > 1e-9
            assert np.array_equal(has[sure], (near < 1.0)[sure])
            second = np.partition(dist, 1, axis=1)[:, 1]
            k = has & (second - near > 1e-9)
            ref = (origin[1 - c] - origin[c]) + x.reshape(2, n, 3)[1 - c][j]
            assert np.abs(q[c * n:(c + 1) * n][k] - ref[k]).max(initial=0.0) <= (1e-6 if precision == "fp32" else 1e-12)
            found += int(has.sum())
    assert found > 1000
