"""The step's and the products' loops at edges of their workgroup: one vertex more than a pass of
eight waves, and banded and whole-range BF16 products of a mesh whose rows are staged in two
chunks, some column blocks' bands lying in one of them.  Bounds as in test_gpu_eval_edges.py and
test_gpu_tile_products.py."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle.model as om
import oracle.step as ostep
from rbc_inputs import meshes
from test_gpu_net_resident import cells_of, polar_mesh
from test_gpu_parity import DT, T, make, oracle_step, rounded, run_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,tol", [("fp32", 2e-5), ("fp64", 1e-11)])
def test_eval_one_vertex_past_eight_waves(precision, tol):
    from paper_1903_06479_amd import Batch
    X, Tr = polar_mesh(7, 73)
    n, m = len(X), om.Model(X, Tr, om.Material(), DT)
    assert n == 513
    x, v, f = (rounded(a, precision) for a in cells_of(X, 2, 5))
    u = rounded(2e-3 * np.random.default_rng(6).standard_normal(x.shape), precision)
    plan = make([(X, Tr)], precision)
    dt = plan.torch_dtype
    grad, terms = Batch(plan, np.zeros(2, np.int32)).eval(T(x, dt), T(v, dt), T(f, dt), T(u, dt))
    grad, terms = grad.cpu().numpy().astype(np.float64), terms.cpu().numpy()
    for c in range(2):
        s = slice(c * n, (c + 1) * n)
        obj = ostep.Objective(m, x[s], v[s], f[s])
        g, gr, noise = obj(x[s] + u[s])
        w = obj.y - obj.x_n                 # the plan leaves out the inertial term's constant
        g -= 0.5 * np.sum(w * (m.Mt @ w)) / DT ** 2
        mu = m.mass[:, None] * u[s] / DT ** 2
        scale = max(np.abs(mu).max(), np.abs(obj.b).max(), np.abs(gr - mu + obj.b).max())
        assert np.abs(grad[s] - gr).max() <= tol * scale, c
        assert abs(terms[c][0] - g) <= tol * noise, c


@pytest.mark.parametrize("precision,tol", [("fp32", 1e-5), ("fp64", 1e-10)])
@pytest.mark.parametrize("lbfgs_m", [2, 5])
def test_step_one_vertex_past_eight_waves(lbfgs_m, precision, tol):
    X, Tr = polar_mesh(7, 73)
    n, m = len(X), om.Model(X, Tr, om.Material(), DT)
    x, v, f = (rounded(a, precision) for a in cells_of(X, 2, 7))
    extra = dict(tol=1e-10, noise_factor=64.0) if precision == "fp64" else {}
    plan = make([(X, Tr)], precision, lbfgs_m=lbfgs_m, max_iter=200, **extra)
    xo, _, st, _ = run_step(plan, np.zeros(2, np.int32), x, v, f)
    for c in range(2):
        s = slice(c * n, (c + 1) * n)
        xr, _, _ = oracle_step(m, x[s], v[s], f[s])
        assert np.abs(xo[s] - xr).max() <= tol * np.ptp(X[:, 0]), (c, st)


@pytest.mark.parametrize("which", [0, 1])
@pytest.mark.parametrize("bf16", [1, 2])
def test_products_in_two_chunks(bf16, which):
    """1026 vertices: 1056 columns staged 672 at a time."""
    X, Tr = meshes.rbc_mesh(1026)
    n, m = len(X), om.Model(X, Tr, om.Material(), DT)
    plan = make([(X, Tr)], "fp32", inverse_bf16=bf16)
    A = np.linalg.inv(m.Ht) if which == 0 else DT * DT * np.linalg.inv(m.Mt)
    for rows in (1, 17, 48, 61):
        buf = torch.zeros(rows * plan.n_pad(0) + 1, device="cuda:0")
        q = np.random.default_rng(rows).standard_normal((rows, n)).astype(np.float32)
        for shift in (0, 1):                # rows on a 16-byte boundary, and 4 bytes past one
            a = buf[shift:shift + rows * plan.n_pad(0)].view(rows, -1)
            a.zero_()
            a[:, :n] = T(q, torch.float32)
            out = plan.apply_inverse(0, which, a).cpu().numpy().astype(np.float64)
            qd = q.astype(np.float64)
            off = A - np.diag(np.diag(A))
            bound = n * 2.0 ** -23 * (np.abs(qd) @ np.abs(A)) + 1e-13 + 1.01 * 2.0 ** -7 * (np.abs(qd) @ np.abs(off))
            if bf16 == 2:
                sd = np.sqrt(np.abs(np.diag(A)))
                bound += 1.0001e-4 * (np.abs(qd) @ sd)[:, None] * sd[None]
            assert np.all(np.abs(out[:, :n] - qd @ A) <= bound), (rows, shift)
