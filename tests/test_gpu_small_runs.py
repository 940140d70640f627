"""Runs around the size below which the crop-first instruments without a private
monitor trace one ray per lane instead of compacting survivors: the same rays
either way, so counts agree with the uncompacted shape's and sums to the order
of the atomic additions (at most 2^21 terms a bin, each within 2^-53)."""
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


@pytest.mark.parametrize("n", [1, 1000, 8 * 4 * 256 * 256 - 1, 8 * 4 * 256 * 256, 8 * 4 * 256 * 256 + 65])
def test_compacting_threshold(torch_cuda, n):
    import paper_2410_08747_amd as m
    announce("compacting threshold", n)
    I = m.Instrument(workloads.basic_absorber())
    assert I.launch_shape[1] == 1
    got = I.run(n, seed=4)[0]
    I.launch_shape = (0, 0, 0, 0)
    ref = I.run(n, seed=4)[0]
    torch_cuda.cuda.synchronize()
    assert np.array_equal(got["count"].cpu().numpy(), ref["count"].cpu().numpy())
    for k in ("sum_w", "sum_w2"):
        g, r = got[k].cpu().numpy(), ref[k].cpu().numpy()
        assert np.all(np.abs(g - r) <= 2.0 ** -32 * np.abs(r)), k
