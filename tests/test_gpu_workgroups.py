"""A cell's step gives the same bits whatever batch it is in: workgroups of four waves (more
tiles than CUs, half a CU's LDS each) and of eight, vectors in LDS and in the workspace
(a batch with a larger mesh), any tile size, default and other histories, optional terms."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_eval_edges import mesh_of
from test_gpu_net_resident import cells_of, polar_mesh
from test_gpu_parity import DT, T

pytestmark = pytest.mark.gpu


def plan_of(ms, optional, **prm):
    from paper_1903_06479_amd import Mesh, Plan, default_material, default_params
    mat = default_material(k_area_global=20.0 if optional else 0.0)
    params = default_params(precision="fp32", volume_normaliser=int(optional), max_iter=12, **prm)
    return Plan([Mesh(*m) for m in ms], DT, material=mat, params=params)


def run(plan, cm, x, v, f, tile):
    from paper_1903_06479_amd import Batch
    b = Batch(plan, np.asarray(cm, np.int32))
    s = b.schedule(cells_per_tile=tile)
    xo, vo, st = b.step(x, v, f)
    torch.cuda.synchronize()
    return s, xo, vo, st.view(torch.uint8)


@pytest.mark.parametrize("mesh,bf16,lbfgs_m,optional", [("42", 0, 5, False), ("pass", 2, 2, False), ("642", 2, 2, False),
                                                        ("642", 1, 5, False), ("642", 0, 8, True), ("742", 2, 2, False),
                                                        ("742", 0, 5, True), ("258", 0, 1, True), ("162", 2, 0, False)])
def test_bits_do_not_depend_on_the_workgroup(mesh, bf16, lbfgs_m, optional):
    m = polar_mesh(20, 37) if mesh == "742" else mesh_of(mesh)     # 742: gradient in the workspace
    n, cells = len(m[0]), 300
    big = mesh_of("2562")
    x, v, f = (T(a, torch.float32) for a in cells_of(m[0], cells, 31))
    plan = plan_of([m], optional, inverse_bf16=bf16, lbfgs_m=lbfgs_m)
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    ref = run(plan, np.zeros(cells), x, v, f, 1)
    assert cells > cu and ref[0]["grid_blocks"] == ref[0]["n_tiles"] == cells           # two workgroups per CU: four waves
    for tile in (3, 21):
        got = run(plan, np.zeros(cells), x, v, f, tile)
        assert got[0]["n_tiles"] <= cu                                                  # eight waves
        assert all(torch.equal(a, b) for a, b in zip(got[1:], ref[1:])), tile
    few = run(plan, np.zeros(7), x[:7 * n], v[:7 * n], f[:7 * n], 2)
    assert torch.equal(few[1], ref[1][:7 * n]) and torch.equal(few[2], ref[2][:7 * n])
    if mesh in ("642", "258"):       # among larger cells: the general evaluation
        xb, vb, fb = (T(a, torch.float32) for a in cells_of(big[0], 1, 33))
        mixed = run(plan_of([m, big], optional, inverse_bf16=bf16, lbfgs_m=lbfgs_m), [0] * 7 + [1],
                    torch.cat([x[:7 * n], xb]), torch.cat([v[:7 * n], vb]), torch.cat([f[:7 * n], fb]), 3)
        assert torch.equal(mixed[1][:7 * n], few[1]) and torch.equal(mixed[2][:7 * n], few[2])


@pytest.mark.parametrize("mesh,bf16,lbfgs_m,terms", [("162", 0, 5, ""), ("162", 1, 2, ""), ("162", 2, 8, ""), ("42", 2, 5, ""),
                                                     ("pass", 0, 2, ""), ("162", 2, 5, "area"), ("162", 0, 2, "literal"),
                                                     ("162", 2, 2, "contacts"), ("162", 0, 8, "contacts")])
def test_four_waves_match_oracle(mesh, bf16, lbfgs_m, terms):
    """More tiles than CUs, so that workgroups have four waves: a few of the cells against the
    oracle, 1e-5 of the diameter as for the other FP32 steps."""
    import oracle.model as om
    import oracle.step as ostep
    from paper_1903_06479_amd import Batch, Mesh, Plan, default_material, default_params
    X, Tr = mesh_of(mesh)
    n, cells, ka = len(X), 300, 60.0 if terms == "area" else 0.0
    x, v, f = (a.astype(np.float32).astype(np.float64) for a in cells_of(X, cells, 51))
    plan = Plan([Mesh(X, Tr)], DT, material=default_material(k_area_global=ka),
                params=default_params(precision="fp32", inverse_bf16=bf16, lbfgs_m=lbfgs_m, max_iter=200,
                                      volume_normaliser=int(terms == "literal")))
    batch = Batch(plan, np.zeros(cells, np.int32))
    s = batch.schedule(cells_per_tile=1)
    assert s["grid_blocks"] == s["n_tiles"] == cells > torch.cuda.get_device_properties(0).multi_processor_count
    ts = [T(a, torch.float32) for a in (x, v, f)]
    contacts = None
    if terms == "contacts":          # tangent planes through and just above some of the vertices
        rng = np.random.default_rng(52)
        nn = rng.standard_normal(x.shape)
        nn /= np.linalg.norm(nn, axis=1, keepdims=True)
        nn[rng.random(len(x)) > 0.2] = 0.0
        q = (x + 0.05 * nn * rng.random((len(x), 1))).astype(np.float32).astype(np.float64)
        nn = nn.astype(np.float32).astype(np.float64)
        contacts, w = (q, nn), 2.0e4
        xo, _, _ = batch.step_contacts(*ts, T(q, torch.float32), T(nn, torch.float32), w)
        batch.schedule(cells_per_tile=3)
        eight, _, _ = batch.step_contacts(*ts, T(q, torch.float32), T(nn, torch.float32), w)
        assert torch.equal(eight, xo)
    else:
        xo, _, _ = batch.step(*ts)
    torch.cuda.synchronize()
    xo = xo.cpu().numpy().astype(np.float64)
    m = om.Model(X, Tr, om.Material(k_area_global=ka), DT)
    for c in (0, 151, 299):
        k = slice(c * n, (c + 1) * n)
        extra = {"contacts": (contacts[0][k], contacts[1][k], w)} if contacts else {}
        xr, _, _ = ostep.step(m, x[k], v[k], f[k], ostep.Params(tol=1e-12, polish=True), literal=terms == "literal", **extra)
        assert np.abs(xo[k] - xr).max() <= 1e-5 * np.ptp(X[:, 0]), c


@pytest.mark.parametrize("lbfgs_m,optional", [(2, False), (5, True)])
def test_bits_in_fp64_do_not_depend_on_the_batch(lbfgs_m, optional):
    from paper_1903_06479_amd import Mesh, Plan, default_material, default_params
    small, big = mesh_of("642"), mesh_of("1026")                   # 1026: gradient and chunks in the workspace
    n, cells = len(small[0]), 7

    def plan(*ms):
        return Plan([Mesh(*m) for m in ms], DT, material=default_material(k_area_global=20.0 if optional else 0.0),
                    params=default_params(precision="fp64", volume_normaliser=int(optional), max_iter=12, lbfgs_m=lbfgs_m))

    x, v, f = (T(a, torch.float64) for a in cells_of(small[0], cells, 31))
    ref = run(plan(small), np.zeros(cells), x, v, f, 1)
    for tile in (3, 7):
        got = run(plan(small), np.zeros(cells), x, v, f, tile)
        assert all(torch.equal(a, b) for a, b in zip(got[1:], ref[1:])), tile
    xb, vb, fb = (T(a, torch.float64) for a in cells_of(big[0], 1, 33))
    mixed = run(plan(small, big), [0] * cells + [1], torch.cat([x, xb]), torch.cat([v, vb]), torch.cat([f, fb]), 3)
    assert torch.equal(mixed[1][:cells * n], ref[1]) and torch.equal(mixed[2][:cells * n], ref[2])
