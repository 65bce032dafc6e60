"""The global-area term's energy is formed from the total area that its gradient is formed
from, summed in FP64 from the FP64 edges: the reported total area has no FP32 rounding in
it (bound 1e-12 of the area: a few FP64 roundings per triangle), in FP32 plans too."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_eval_edges import mesh_of
from test_gpu_net_resident import cells_of
from test_gpu_parity import DT, T, rounded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mesh", ["258", "642", "1026"])
def test_total_area_of_the_area_term_is_fp64(mesh):
    from paper_1903_06479_amd import Batch, Mesh, Plan, default_material, default_params
    X, Tr = mesh_of(mesh)
    n = len(X)
    x, v, f = (rounded(a, "fp32") for a in cells_of(X, 3, 41))
    u = rounded(2e-3 * np.random.default_rng(42).standard_normal(x.shape), "fp32")
    plan = Plan([Mesh(X, Tr)], DT, material=default_material(k_area_global=20.0), params=default_params(precision="fp32"))
    _, terms = Batch(plan, np.zeros(3, np.int32)).eval(*(T(a, torch.float32) for a in (x, v, f, u)))
    terms = terms.cpu().numpy()
    for c in range(3):
        y = (x + u)[c * n:(c + 1) * n]
        area = 0.5 * np.linalg.norm(np.cross(y[Tr[:, 0]] - y[Tr[:, 2]], y[Tr[:, 1]] - y[Tr[:, 2]]), axis=1).sum()
        assert abs(terms[c][9] - area) <= 1e-12 * area, c
