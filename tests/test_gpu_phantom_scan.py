"""The scan of a phantom at creation (bricks of 4^3 voxels, the last ones cut off by
the volume): an id that the table does not have is found wherever it is, and the
occupied box holds a single voxel wherever it is -- the image then equals the
oracle's, which walks every voxel."""
import numpy as np
import pytest

import oracle
import workloads

from test_gpu_parity import announce, compare_bins

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (4, 4, 4), (5, 6, 7), (9, 3, 8), (64, 64, 64), (33, 65, 68), (130, 7, 12)]


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def places(shape):
    """Corners, and the voxels on both sides of the last whole brick."""
    edge = [sorted({0, n - 1, max(0, n // 4 * 4 - 1), min(n - 1, n // 4 * 4)}) for n in shape]
    rng = np.random.default_rng(sum(shape))
    every = [(z, y, x) for z in edge[0] for y in edge[1] for x in edge[2]]
    return [every[i] for i in rng.permutation(len(every))[:12]]


@pytest.mark.parametrize("shape", SHAPES)
def test_every_voxel_is_scanned(torch_cuda, shape):
    import paper_2410_08747_amd as m
    announce("phantom scan", shape)
    mu = workloads.make_mu_tables(3)
    for place in places(shape):
        vol = np.ones(shape, np.uint8)
        vol[place] = mu.shape[0]
        with pytest.raises(m.MxrError):
            m.Instrument(workloads.edct_projection(vol, mu))
        vol[place] = mu.shape[0] - 1
        m.Instrument(workloads.edct_projection(vol, mu)).close()


@pytest.mark.parametrize("shape", SHAPES)
def test_occupied_box(torch_cuda, shape):
    import paper_2410_08747_amd as m
    announce("occupied box", shape)
    n = 20_000
    for place in places(shape)[:4]:
        vol = np.zeros(shape, np.uint8)
        vol[place] = 6
        ins = workloads.edct_projection(vol, workloads.make_mu_tables(3), angle=0.4, strata=16, nx=24, ny=24, ne=2)
        o = oracle.run(ins, n, seed=3)[0]
        I = m.Instrument(ins)
        for occupancy in (0, 4):
            I.launch_shape = (occupancy, 1, 0, 1)
            got = I.run(n, seed=3)[0]
            torch_cuda.cuda.synchronize()
            compare_bins(got, o, f"{shape} {place} {occupancy}")
