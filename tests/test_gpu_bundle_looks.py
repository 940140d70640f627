"""The bundle walk's looks at layers, where a small feature or the seam between two
chunks of 64 bricks (256 layers) could be lost: long volumes, nearly empty, with
single voxels of other materials -- on the faces and corners of bricks, in the last
brick that the volume cuts off, alone in a chunk's last brick, followed by a uniform
and by another mixed brick -- with more mixed bricks than one look at voxels covers
(16), one in every brick, and with slabs that change every ray's material at once.
Narrow bundles, along the axis and against it, under the exact and the fixed-step
model and for photons scattered once; the form forced to bundles.  Against the run
with a ledger, one ray at a time."""
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


def empty(layers, first=0):
    """Long across z; two voxels make the occupied box span it."""
    vol = np.zeros((layers, 48, 50), np.uint8)
    vol[first, 24, 25] = 2
    vol[-1, 23, 24] = 3
    return vol


def specks(layers, every, first=0, seed=1):
    """A few single voxels in each of every so many layers."""
    vol = empty(layers, first)
    rng = np.random.default_rng(seed)
    for z in range(first, layers, every):
        for _ in range(3):
            vol[z, rng.integers(8, 40), rng.integers(8, 42)] = rng.integers(1, 8)
    return vol


def seam(*layers, first=0):
    """Voxels about the seam of the first two chunks: corners and faces of bricks."""
    vol = empty(300, first)
    for z in layers:
        for y, x in ((24, 24), (23, 23), (27, 20), (20, 27), (31, 30)):
            vol[z, y, x] = 5
    return vol


def slabs():
    """Whole layers of another material, on and off the bricks' faces, and specks."""
    vol = specks(300, 60)
    vol[40:80] = 1
    vol[101:103] = 4
    vol[250:262] = 6
    vol[200, 10:30, 10:30] = 7
    return vol


VOLUMES = {
    "empty 255": lambda: empty(255), "empty 256": lambda: empty(256), "empty 257": lambda: empty(257),
    "specks 64": lambda: specks(64, 7), "specks 300": lambda: specks(300, 40), "specks 17": lambda: specks(300, 8),
    "specks all": lambda: specks(300, 4), "specks off the bricks": lambda: specks(297, 9, first=5),
    "seam, mixed then uniform": lambda: seam(253), "seam, mixed then mixed": lambda: seam(253, 257),
    "seam, uniform then mixed": lambda: seam(256), "seam, last layer": lambda: seam(255),
    "seam, later chunk": lambda: seam(254, 258, first=6), "slabs": slabs,
    "long 600": lambda: specks(600, 37),
}


def check(torch, ins, n, seed, rtol):
    import paper_2410_08747_amd as m
    I = m.Instrument(ins)
    I.launch_shape = (4, 1, 0, 1)
    got, ref = I.run(n, seed=seed)[0], I.run(n, seed=seed, ledger=I.new_ledger())[0]
    torch.cuda.synchronize()
    assert int(ref["count"].sum()) > 1000
    assert np.array_equal(got["count"].cpu().numpy(), ref["count"].cpu().numpy())
    for k in ("sum_w", "sum_w2"):
        g, r = got[k].cpu().numpy(), ref[k].cpu().numpy()
        assert np.all(np.abs(g - r) <= rtol * np.abs(r)), (k, np.max(np.abs(g - r) / np.where(r != 0, r, 1)))


@pytest.mark.parametrize("angle", [0.0, np.pi, 0.02])
@pytest.mark.parametrize("model", [{}, {"step": 1.0 / 3.0}, {"step": 2.5}, {"scatter_order": 1}], ids=["exact", "steps", "long steps", "scattered"])
@pytest.mark.parametrize("name", sorted(VOLUMES))
def test_looks(torch_cuda, name, model, angle):
    announce("bundle looks", name, model, angle)
    mu = workloads.make_mu_tables(3)
    if "scatter_order" in model:
        mu = workloads.make_scatter_tables(mu)
    n, strata = 300_001, 130
    ins = workloads.edct_projection(VOLUMES[name](), mu, angle=angle, strata=strata, nx=30, ny=30, ne=2, **model)
    check(torch_cuda, ins, n, 3, 1e-9 if "scatter_order" in model else 1e-11)


@pytest.mark.parametrize("name", ["specks 17", "seam, mixed then mixed", "specks off the bricks"])
def test_looks_across_x(torch_cuda, name):
    """The same with the long axis along x, which bricks and rows run along."""
    announce("bundle looks, x", name)
    vol = np.ascontiguousarray(np.moveaxis(VOLUMES[name](), 0, 2))
    for angle in (0.5 * np.pi, -0.5 * np.pi):
        for voxel in (1.0, 0.8):
            ins = workloads.edct_projection(vol, workloads.make_mu_tables(3), angle=angle, strata=130, nx=30, ny=30, ne=2)
            ins["components"][1]["voxel"] = voxel
            check(torch_cuda, ins, 300_001, 4, 1e-11)
