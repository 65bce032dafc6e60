"""The schedule that a batch reports is the one it runs: sizes set by hand are kept, also
after the tuner, and a tuned schedule can be given to another batch."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from rbc_inputs import meshes, workloads
from test_gpu_parity import T, make, rounded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [37, 300])
def test_tuned_schedule_is_reported_as_it_is(cells):
    from paper_1903_06479_amd import Batch
    b = workloads.shear(n_cells=cells, seed=24)
    x, v = rounded(b.x, "fp32"), rounded(b.v, "fp32")
    f = rounded(workloads.drag_forces(b, x, v), "fp32")
    plan = make([b.meshes[642]], "fp32", inverse_bf16=2)
    batch, other = (Batch(plan, np.zeros(cells, np.int32)) for _ in range(2))
    xi, vi, fi = (T(a, torch.float32) for a in (x, v, f))
    best = batch.autotune(xi, vi, fi)
    tuned = batch.schedule()
    assert tuned["n_tiles"] == -(-cells // tuned["cells_per_tile"]) and best["tile_cells"] == tuned["cells_per_tile"]
    assert other.schedule(tuned["cells_per_tile"], tuned["lbfgs_m"]) == tuned
    assert batch.schedule(lbfgs_m=1) == dict(tuned, lbfgs_m=1)
    for tile in (best["cells_per_tile"], 5, 1):
        s = batch.schedule(cells_per_tile=tile)
        assert s["cells_per_tile"] == tile and s["n_tiles"] == -(-cells // tile)


@pytest.mark.parametrize("precision,n,cells,tile", [("fp64", 1026, 2900, 4), ("fp64", 642, 4600, 5), ("fp32", 642, 4600, 5),
                                                    ("fp32", 1026, 2900, 6), ("fp32", 2562, 40, 1)])
def test_default_tiles_weigh_the_products(precision, n, cells, tile):
    """Dense products, which grow like n^2 and take a second or third pass where the tile's
    rows exceed the LDS: the default stays with the size that shares them without that."""
    from paper_1903_06479_amd import Batch
    b = workloads.shear(n_cells=1, seed=1)
    mesh = b.meshes[642] if n == 642 else meshes.rbc_mesh(n)
    assert Batch(make([mesh], precision), np.zeros(cells, np.int32)).schedule()["cells_per_tile"] == tile
