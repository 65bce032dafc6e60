"""The tile products at the edges of their blocks: fewer column blocks than waves, rows that
fill one to four row blocks with remainders, rows staged in LDS or not, bands whose blocks
hold fewer operands than a batch, and k' ranges cut into chunks.  Bounds: the rounding of the
sums, n eps times the sum of the terms' magnitudes (FP32 sums of n_pad terms in any order),
plus 1.01 2^-7 of the off-diagonal terms for BF16 products (both factors are rounded to
within 2^-8), plus what the band may drop (entries below 1e-4 sqrt(A_ii A_jj))."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle.model as om
from test_gpu_eval_edges import mesh_of
from test_gpu_parity import DT, T, make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 16, 17, 33, 48, 61])
@pytest.mark.parametrize("precision,bf16", [("fp32", 0), ("fp64", 0), ("fp32", 1), ("fp32", 2)])
@pytest.mark.parametrize("mesh", ["12", "42", "poles"])
def test_apply_inverse_at_block_edges(mesh, precision, bf16, rows):
    X, Tr = mesh_of(mesh)
    n, m = len(X), om.Model(X, Tr, om.Material(), DT)
    plan = make([(X, Tr)], precision, inverse_bf16=bf16)
    q = np.zeros((rows, plan.n_pad(0)))
    q[:, :n] = np.random.default_rng(rows).standard_normal((rows, n)).astype(np.float32)
    out = plan.apply_inverse(0, 0, T(q, plan.torch_dtype)).cpu().numpy().astype(np.float64)
    A = np.linalg.inv(m.Ht)
    q = q[:, :n]
    bound = n * (2.0 ** -23 if precision == "fp32" else 2.0 ** -52) * (np.abs(q) @ np.abs(A)) + 1e-13
    if precision == "fp64":
        bound *= np.linalg.cond(A)                      # the two inverses' own rounding
    if bf16:
        off = A - np.diag(np.diag(A))
        bound += 1.01 * 2.0 ** -7 * (np.abs(q) @ np.abs(off))
    if bf16 == 2:
        sd = np.sqrt(np.diag(A))
        bound += 1.0001e-4 * (np.abs(q) @ sd)[:, None] * sd[None]
    assert np.all(np.abs(out[:, :n] - q @ A) <= bound)


@pytest.mark.parametrize("precision,bf16", [("fp32", 0), ("fp64", 0), ("fp32", 1), ("fp32", 2)])
@pytest.mark.parametrize("mesh", ["42", "642"])
def test_step_is_the_same_for_every_tile_size(mesh, precision, bf16):
    """One cell's result does not depend on the rows around it: 22 cells in tiles of 1 to 21
    (one to four row blocks; staged and not) give the same bits."""
    from paper_1903_06479_amd import Batch
    from test_gpu_net_resident import cells_of
    X, Tr = mesh_of(mesh)
    plan = make([(X, Tr)], precision, inverse_bf16=bf16)
    dt = plan.torch_dtype
    x, v, f = (T(a, dt) for a in cells_of(X, 22, 9))
    batch = Batch(plan, np.zeros(22, np.int32))
    ref = None
    for tile in (1, 5, 6, 11, 16, 21):
        batch.schedule(cells_per_tile=tile)
        xo, vo, _ = batch.step(x, v, f)
        torch.cuda.synchronize()
        if ref is not None:
            assert torch.equal(xo, ref[0]) and torch.equal(vo, ref[1]), tile
        ref = (xo, vo)


@pytest.mark.parametrize("precision,cells,tile,tiles", [("fp32", 3, 1, 3), ("fp64", 3, 1, 3), ("fp32", 1100, 3, 367),
                                                        ("fp64", 1000, 4, 250)])
def test_default_tiles_fill_the_workgroups(precision, cells, tile, tiles):
    """Few cells are spread over the workgroups (two per compute unit in FP32, one for an
    FP64 batch of 642 vertices; 256 units); an explicit size is kept."""
    from paper_1903_06479_amd import Batch
    X, Tr = mesh_of("642")
    batch = Batch(make([(X, Tr)], precision, inverse_bf16=2 if precision == "fp32" else 0), np.zeros(cells, np.int32))
    assert batch.schedule()["cells_per_tile"] == tile and batch.schedule()["n_tiles"] == tiles
    assert batch.schedule(cells_per_tile=5)["n_tiles"] == (cells + 4) // 5
