"""Where a training epoch keeps its batches' weight sums: a batch's rows weigh
omega_i / sum omega, so batches of one row do not depend on omega at all, and
doubling every omega changes nothing, bit for bit.  More steps than one launch
sums, and batches whose partial gradients fill their region of the workspace."""
import math

import numpy as np
import pytest

import workloads

from test_gpu_parity import announce

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def train(torch, rows, batch, omega):
    import paper_2410_08747_amd as m
    rng = np.random.default_rng(3)
    net = m.ProposalNet(workloads.init_mlp_params(3), batch=batch)
    ctx = torch.tensor(rng.normal(0.0, 1.0, (rows, 6)), dtype=torch.float32, device="cuda")
    t = math.tan(workloads.edct_half_angle())
    y = torch.tensor(np.stack([rng.uniform(-t, t, rows), rng.uniform(-t, t, rows), rng.uniform(21.0, 149.0, rows)], 1),
                     device="cuda")
    log = torch.empty(-(-rows // batch), dtype=torch.float64, device="cuda")
    net.train(ctx, y, torch.tensor(omega, device="cuda"), (-t, -t, 20.0), (t, t, 150.0), epochs=1, lr=1e-4, loss_log=log)
    torch.cuda.synchronize()
    return log.cpu().numpy(), net.master.cpu().numpy()


@pytest.mark.parametrize("rows,batch", [(5, 1), (12_400, 1), (300, 7), (80_003, 40_000), (70_001, 32_513)])
def test_weights_are_relative(torch_cuda, rows, batch):
    announce("training, weight sums", rows, batch)
    omega = np.random.default_rng(4).uniform(0.1, 2.0, rows)
    one = train(torch_cuda, rows, batch, omega)
    for other in ([2.0 * omega] if batch > 1 else [2.0 * omega, omega[::-1].copy()]):
        two = train(torch_cuda, rows, batch, other)
        assert np.all(np.isfinite(one[0])) and np.array_equal(one[0], two[0]) and np.array_equal(one[1], two[1])
