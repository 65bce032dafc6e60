"""Minibatches that fill the memory: one that the any-size kernels hold and the resident ones do not
(they keep two fifths more per cell) still gives its gradient, and smaller ones after it run as
before.  The minibatch repeats the cells of a small batch, so the gradient is known: bound 1e-3
as for the two kernels elsewhere."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle.mpnn as mp
from rbc_inputs import meshes
from test_gpu_net import T, gpu_params, make

pytestmark = pytest.mark.gpu


def test_minibatch_beyond_the_resident_kernels_memory():
    from paper_1903_06479_amd import Batch, Net
    X, Tr = meshes.rbc_mesh(642)
    cells, g = 256, torch.Generator(device="cuda:0").manual_seed(3)
    plan = make([(X, Tr)], "fp32")
    batch = Batch(plan, np.zeros(cells, np.int32))
    x = T(X).repeat(cells, 1)
    x, v, f, d = (a + s * torch.randn(x.shape, generator=g, device=x.device) for a, s in ((x, 0.05), (0, 0.01), (0, 3.0), (0, 1e-3)))
    u0 = batch.first_guess(x, v, f)
    x_next = x + u0 + d
    net = Net(plan, gpu_params(mp.NetConfig(), 17).astype(np.float32))
    loss, grad = net.loss_grad(batch, x, v, f, x_next, u0)
    grad = grad.clone()
    np_, planes = plan.n_pad(0), mp.NetConfig().layers + 1
    per_cell = np_ * (2 * 32 + 2 * planes * 2 * 64 + 2 * 12) + 168          # any-size kernels, bytes
    torch.cuda.empty_cache()
    times = int(0.9 * torch.cuda.mem_get_info()[0] / per_cell) // cells
    pick = (torch.arange(times * cells, device=x.device) % cells).int()
    assert (per_cell + np_ * (planes - 1) * 2 * 64) * times * cells > torch.cuda.mem_get_info()[0]
    big, gb = net.loss_grad(batch, x, v, f, x_next, u0, cells=pick)
    assert abs(big - loss) <= 1e-3 * loss and float((gb - grad).norm() / grad.norm()) <= 1e-3
    again, ga = net.loss_grad(batch, x, v, f, x_next, u0)
    assert again == loss and torch.equal(ga, grad)
