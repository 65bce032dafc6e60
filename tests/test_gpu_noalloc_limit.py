"""The allocation-free step takes the largest workspace of a workgroup that it ever took: 21 FP64
cells of 6,602 vertices with a history of seven (64 MiB before the step kept x_n with its
vectors, 67.2 MiB with it)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_net_resident import polar_mesh
from test_gpu_parity import T, make

pytestmark = pytest.mark.gpu


def test_noalloc_step_takes_the_largest_workgroup():
    from paper_1903_06479_amd import Batch, CELL_STATS_DTYPE
    m = polar_mesh(100, 66)
    plan = make([m], "fp64", lbfgs_m=7, cells_per_tile=21, max_iter=2)
    batch = Batch(plan, np.zeros(21, np.int32))
    rng = np.random.default_rng(3)
    x = T(np.tile(m[0], (21, 1)) + 1e-3 * rng.standard_normal((21 * len(m[0]), 3)), torch.float64)
    v, f = torch.zeros_like(x), T(rng.standard_normal(x.shape), torch.float64)
    st = torch.empty(21 * CELL_STATS_DTYPE.itemsize, dtype=torch.uint8, device=x.device)
    xr, vr, _ = batch.step(x, v, f)
    xo, vo = torch.empty_like(x), torch.empty_like(x)
    batch.step_noalloc(x, v, f, xo, vo, stats=st)
    torch.cuda.synchronize()
    assert torch.equal(xo, xr) and torch.equal(vo, vr)
