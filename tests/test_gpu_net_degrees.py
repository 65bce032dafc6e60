"""The LDS-resident network on meshes with a few vertices of high degree, against the kernels
that gather from memory: the results, and the time, which follows the row blocks that hold
such vertices and not the whole mesh (bound: six times the time of the same rows at degree six;
one list length for all rows took twelve, the row blocks' own three)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle.mpnn as mp
from rbc_inputs import meshes
from test_gpu_net import T, gpu_params, make, relerr
from test_gpu_net_resident import cells_of, polar_mesh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("segments,rings", [(20, 30), (200, 3)])
def test_high_degrees_match_the_any_size_kernels(segments, rings, monkeypatch):
    from paper_1903_06479_amd import Batch, Net
    m = polar_mesh(segments, rings)
    count, theta = 5, gpu_params(mp.NetConfig(), 17).astype(np.float32)
    plan = make([m], "fp64")
    batch = Batch(plan, np.zeros(count, np.int32))
    xs = [T(a, torch.float64) for a in cells_of(m[0], count, 18)]
    u0 = batch.first_guess(*xs)
    x_next = xs[0] + u0 + 1e-3 * torch.randn(u0.shape, dtype=torch.float64, device=u0.device,
                                              generator=torch.Generator(device=u0.device).manual_seed(19))
    out = []
    for env in (False, True):
        if env:
            monkeypatch.setenv("NPFEM_NET_NO_LDS", "1")
        net = Net(plan, theta)
        loss, g = net.loss_grad(batch, *xs, x_next, u0)
        out.append((loss, g.cpu().numpy().astype(np.float64), net.infer(batch, *xs).cpu().numpy()))
    assert abs(out[0][0] - out[1][0]) <= 1e-3 * out[1][0]
    assert relerr(out[0][1], out[1][1]) <= 1e-3
    assert relerr(out[0][2], out[1][2]) <= 1e-3


def test_time_follows_the_rows_of_high_degree():
    from paper_1903_06479_amd import Batch, Net
    count, theta, us = 2000, gpu_params(mp.NetConfig(), 17).astype(np.float32), []
    for m in (meshes.rbc_mesh(642), polar_mesh(200, 3)):
        plan = make([m], "fp32")
        batch, net = Batch(plan, np.zeros(count, np.int32)), Net(plan, theta)
        x = T(m[0]).repeat(count, 1)
        v, f = 0.01 * torch.randn_like(x), torch.randn_like(x)
        net.infer(batch, x, v, f)
        best = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            net.infer(batch, x, v, f)
            b.record()
            torch.cuda.synchronize()
            best.append(a.elapsed_time(b))
        us.append(min(best))
    assert us[1] <= 6 * us[0], us


@pytest.mark.parametrize("segments,rings,cells", [(20, 37, 60), (16, 40, 60), (200, 3, 60), (11, 31, 60)])
def test_features_keep_their_precision(segments, rings, cells, monkeypatch):
    """Meshes above 704 rows or of high degree form their features in FP64, as the kernels that
    gather from memory do: the same features are rounded to BF16, and the corrections are the
    same bits (features formed in FP32 round the other way in a few of a cell's)."""
    from paper_1903_06479_amd import Batch, Net
    m = polar_mesh(segments, rings)
    theta = gpu_params(mp.NetConfig(), 17).astype(np.float32)
    plan = make([m], "fp32")
    batch = Batch(plan, np.zeros(cells, np.int32))
    xs = [T(a) for a in cells_of(m[0], cells, 20)]
    got = Net(plan, theta).infer(batch, *xs).clone()
    monkeypatch.setenv("NPFEM_NET_NO_LDS", "1")
    ref = Net(plan, theta).infer(batch, *xs)
    torch.cuda.synchronize()
    assert torch.equal(got, ref)
