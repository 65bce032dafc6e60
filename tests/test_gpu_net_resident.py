"""The LDS-resident network kernels at the edges of their ranges (few rows, part-filled row
blocks, four and eight waves, vertices of high degree, mixed meshes in one minibatch)
against the FP64 oracle and the any-size kernels.  Bounds: 1e-2 in the relative L2 norm as
for the network's other tests (about ten BF16 roundings of at most 2^-9 along a path, in
quadrature); against the any-size kernels, which round at the same places, 1e-3 (a sum taken
in another order moves at most single BF16 roundings)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle.model as om
import oracle.mpnn as mp
from rbc_inputs import meshes, workloads
from test_gpu_net import DT, REL, T, gpu_params, make, relerr

pytestmark = pytest.mark.gpu


def polar_mesh(segments, rings):
    """A sphere of `rings` circles of `segments` vertices and two poles of that degree."""
    th = np.pi * np.arange(1, rings + 1) / (rings + 1)
    ph = 2 * np.pi * np.arange(segments) / segments
    v = [[0.0, 0.0, 1.0]] + [[np.sin(a) * np.cos(p), np.sin(a) * np.sin(p), np.cos(a)] for a in th for p in ph]
    v.append([0.0, 0.0, -1.0])
    t, at = [], lambda r, s: 1 + r * segments + s % segments
    for s in range(segments):
        t += [[0, at(0, s), at(0, s + 1)], [len(v) - 1, at(rings - 1, s + 1), at(rings - 1, s)]]
        for r in range(rings - 1):
            t += [[at(r, s), at(r + 1, s), at(r + 1, s + 1)], [at(r, s), at(r + 1, s + 1), at(r, s + 1)]]
    return 3.0 * np.array(v), np.array(t, np.int32)


def cells_of(X, count, seed):
    rng = np.random.default_rng(seed)
    x = np.concatenate([X @ workloads.random_rotation(rng).T + 0.05 * rng.standard_normal(X.shape) for _ in range(count)])
    return x, 0.01 * rng.standard_normal(x.shape), 3.0 * rng.standard_normal(x.shape)


@pytest.mark.parametrize("mesh", ["12", "42", "66", "162", "258", "642", "poles"])
def test_resident_network_matches_oracle(mesh):
    """Inference (FP32 inputs) and the training gradient (FP64 inputs) of a few cells."""
    from paper_1903_06479_amd import Batch, Net
    X, Tr = polar_mesh(11, 31) if mesh == "poles" else meshes.rbc_mesh(int(mesh)) if int(mesh) > 12 else \
        meshes.sphere_mesh(12, 3.0)
    m = om.Model(X, Tr, om.Material(), DT)
    n, count, cfg = len(X), 5, mp.NetConfig()
    x, v, f = (a.astype(np.float32).astype(np.float64) for a in cells_of(X, count, 3))
    theta = gpu_params(cfg, 11)
    A = mp.neighbour_mean_matrix(n, Tr)
    p32 = make([(X, Tr)], "fp32")
    net = Net(p32, theta.astype(np.float32))
    b32 = Batch(p32, np.zeros(count, np.int32))
    delta = net.infer(b32, T(x), T(v), T(f)).cpu().numpy().astype(np.float64)
    p64 = make([(X, Tr)], "fp64")
    net64, b64 = Net(p64, theta.astype(np.float32)), Batch(p64, np.zeros(count, np.int32))
    xs = [T(a, torch.float64) for a in (x, v, f)]
    u0 = b64.first_guess(*xs)
    x_next = x + u0.cpu().numpy() + 1e-3 * np.random.default_rng(5).standard_normal(x.shape)
    pick = np.array([3, 0, 4], np.int32)
    loss, grad = net64.loss_grad(b64, *xs, T(x_next, torch.float64), u0, cells=T(pick, torch.int32))
    data = []
    for c in range(count):
        s = slice(c * n, (c + 1) * n)
        feats, R, sc = mp.features(X, x[s], v[s], f[s], m.mass, DT, cfg)
        o, _ = mp.forward(theta, feats, A, cfg)
        assert relerr(delta[s], sc * (o @ R.T)) <= REL, c
        if c in pick:
            data.append((feats, mp.target(R, sc, x_next[s] - x[s] - u0.cpu().numpy()[s])))
    lr, gr = mp.loss_and_grad(theta, data, A, cfg)
    assert abs(loss - lr) <= REL * lr
    assert relerr(grad.cpu().numpy().astype(np.float64), gr) <= REL


def test_mixed_minibatch_matches_the_any_size_kernels(monkeypatch):
    """A minibatch of 258- and 642-vertex cells, more cells than gradient slots: gradient and
    inference of the resident kernels against those that gather from memory."""
    from paper_1903_06479_amd import Batch, Net
    b = workloads.uneven(n_cells=100, seed=51, sizes=(258, 642), counts=(0.5, 0.5))
    sizes = sorted(b.meshes)
    cm = np.array([sizes.index(int(k)) for k in b.cell_nverts], np.int32)
    rng = np.random.default_rng(52)
    v = 0.01 * rng.standard_normal(b.x.shape)
    f = workloads.drag_forces(b, b.x, v)
    theta = gpu_params(mp.NetConfig(), 13).astype(np.float32)
    plan = make([b.meshes[k] for k in sizes], "fp64")
    batch = Batch(plan, cm)
    xs = [T(a, torch.float64) for a in (b.x, v, f)]
    u0 = batch.first_guess(*xs)
    x_next = xs[0] + u0 + T(1e-3 * rng.standard_normal(b.x.shape), torch.float64)
    pick = T(rng.permutation(100)[:90].astype(np.int32), torch.int32)
    out = []
    for env in (False, True):
        if env:
            monkeypatch.setenv("NPFEM_NET_NO_LDS", "1")
        net = Net(plan, theta)
        loss, g = net.loss_grad(batch, *xs, x_next, u0, cells=pick)
        out.append((loss, g.cpu().numpy().astype(np.float64), net.infer(batch, *xs).cpu().numpy()))
    assert abs(out[0][0] - out[1][0]) <= 1e-3 * out[1][0]
    assert relerr(out[0][1], out[1][1]) <= 1e-3
    assert relerr(out[0][2], out[1][2]) <= 1e-3
