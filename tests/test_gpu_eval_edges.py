"""The evaluation and the step at the edges of their loops: few vertices (waves without
work), one more vertex than a pass of the workgroup, vertices of high degree (several groups
of the neighbour and corner lists, with padding), and the longest and shortest histories (more
and fewer sums than one reduction holds).  Bounds as in test_gpu_parity.py: the rounding of
the largest terms for one evaluation, 1e-5 (FP32) and 1e-10 (FP64) cell diameters for a step."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle.model as om
import oracle.step as ostep
from rbc_inputs import meshes
from test_gpu_net_resident import cells_of, polar_mesh
from test_gpu_parity import DT, T, make, oracle_step, rounded, run_step

pytestmark = pytest.mark.gpu


def mesh_of(name):
    if name == "poles":                      # 343 vertices, two of degree 11
        return polar_mesh(11, 31)
    if name == "pass":                       # 257 vertices: one more than the workgroup's threads
        return polar_mesh(15, 17)
    return meshes.rbc_mesh(int(name)) if int(name) > 12 else meshes.sphere_mesh(12, 3.0)


@pytest.mark.parametrize("precision,tol", [("fp32", 2e-5), ("fp64", 1e-11)])
@pytest.mark.parametrize("mesh", ["12", "42", "pass", "poles"])
def test_eval_at_loop_edges(mesh, precision, tol):
    from paper_1903_06479_amd import Batch
    X, Tr = mesh_of(mesh)
    n, m = len(X), om.Model(X, Tr, om.Material(), DT)
    x, v, f = (rounded(a, precision) for a in cells_of(X, 3, 5))
    u = rounded(2e-3 * np.random.default_rng(6).standard_normal(x.shape), precision)
    plan = make([(X, Tr)], precision)
    dt = plan.torch_dtype
    grad, terms = Batch(plan, np.zeros(3, np.int32)).eval(T(x, dt), T(v, dt), T(f, dt), T(u, dt))
    grad, terms = grad.cpu().numpy().astype(np.float64), terms.cpu().numpy()
    for c in range(3):
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
@pytest.mark.parametrize("mesh,lbfgs_m", [("42", 8), ("pass", 1), ("pass", 8), ("poles", 2)])
def test_step_at_loop_edges(mesh, lbfgs_m, precision, tol):
    X, Tr = mesh_of(mesh)
    n, m = len(X), om.Model(X, Tr, om.Material(), DT)
    x, v, f = (rounded(a, precision) for a in cells_of(X, 3, 7))
    extra = dict(tol=1e-10, noise_factor=64.0) if precision == "fp64" else {}
    plan = make([(X, Tr)], precision, lbfgs_m=lbfgs_m, max_iter=200, **extra)
    xo, _, st, _ = run_step(plan, np.zeros(3, np.int32), x, v, f)
    for c in range(3):
        s = slice(c * n, (c + 1) * n)
        xr, _, _ = oracle_step(m, x[s], v[s], f[s])
        assert np.abs(xo[s] - xr).max() <= tol * np.ptp(X[:, 0]), (c, st)
