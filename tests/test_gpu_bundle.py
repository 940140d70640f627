"""The wave-wide walk of plain runs (footprints of 64 layers at a time, then
only the layers where the bundle meets a boundary) against the event walk
that runs with a ledger take: counts equal, sums within the per-bin parity bar
divided by a hundred.  Volumes, voxel sizes, angles and strata are chosen
where the footprints can go wrong: layer counts around the 64 of a chunk,
volumes where every layer is mixed, one voxel, one material, thin and long
volumes (one axis beyond the bundle's limit), a corner material that is not
air, waves whose rays differ in dominant axis or direction, bundles from a
fraction of a voxel to many voxels wide, and rays that run along an axis."""
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


def noise(shape, seed=1):
    return np.random.default_rng(seed).integers(0, 8, shape).astype(np.uint8)


def slabs(shape, axis):
    """Layers of changing material across one axis, three voxels thick."""
    idx = np.indices(shape)[axis]
    return ((idx // 3) % 5).astype(np.uint8)


def shell(shape):
    vol = np.full(shape, 3, np.uint8)  # the corner's material is not air
    vol[4:-4, 4:-4, 4:-4] = 0
    vol[10:-10, 9:-11, 8:-9] = 5
    return vol


VOLUMES = {
    "noise 33": lambda: noise((33, 33, 33)),
    "noise 64x65x63": lambda: noise((64, 65, 63)),
    "slabs z 128": lambda: slabs((128, 40, 50), 0),
    "slabs x 129": lambda: slabs((40, 50, 129), 2),
    "shell 70": lambda: shell((70, 71, 72)),
    "one voxel": lambda: np.full((1, 1, 1), 4, np.uint8),
    "one material": lambda: np.full((20, 30, 40), 2, np.uint8),
    "one odd voxel": lambda: np.where(np.arange(50 ** 3).reshape(50, 50, 50) == 60000, 6, 1).astype(np.uint8),
    "thin plate": lambda: noise((1, 90, 90)),
    "long": lambda: noise((4, 4, 2500)),
    "luggage 96": lambda: workloads.make_phantom(96, seed=4),
}
VIEWS = [(0.0, 1.0, 256, 300_001), (0.7853981, 1.0, 16, 120_007), (3.2, 0.75, 64, 200_003), (1.5707963267948966, 1.3, 4, 50_021)]


@pytest.mark.parametrize("view", range(len(VIEWS)))
@pytest.mark.parametrize("name", sorted(VOLUMES))
def test_bundle_image_equals_the_event_walks(torch_cuda, name, view):
    import paper_2410_08747_amd as m
    angle, voxel, strata, n = VIEWS[view]
    announce("bundle walk", name, VIEWS[view])
    ins = workloads.edct_projection(VOLUMES[name](), workloads.make_mu_tables(3), angle=angle, strata=strata, nx=64, ny=32,
                                    ne=4)
    ins["components"][1]["voxel"] = voxel
    I = m.Instrument(ins)
    got, ref = I.run(n, seed=8)[0], I.run(n, seed=8, ledger=I.new_ledger())[0]
    torch_cuda.cuda.synchronize()
    assert int(ref["count"].sum()) > 1000
    assert np.array_equal(got["count"].cpu().numpy(), ref["count"].cpu().numpy())
    for k in ("sum_w", "sum_w2"):
        g, r = got[k].cpu().numpy(), ref[k].cpu().numpy()
        assert np.array_equal(g == 0, r == 0)
        assert np.all(np.abs(g - r) <= 1e-11 * np.abs(r)), (k, np.max(np.abs(g - r) / np.where(r != 0, r, 1)))


@pytest.mark.parametrize("place", ["inside", "beside", "along the axis"])
def test_bundles_from_other_places(torch_cuda, place):
    """A source inside the volume (paths start there, in every direction of a
    wide cone), beside it, and one whose cone is a pencil along an axis."""
    import paper_2410_08747_amd as m
    announce("bundle walk", place)
    ins = workloads.edct_projection(noise((60, 62, 66), 5), workloads.make_mu_tables(3), angle=0.0, strata=32, nx=32, ny=16,
                                    ne=4)
    src, ph, det = ins["components"]
    if place == "inside":
        ph["pos"], src["half_angle"] = (3.0, -2.0, 5.0), 1.2
        det.update(pos=(0.0, 0.0, 60.0), xmin=-100.0, xmax=100.0, ymin=-100.0, ymax=100.0)
    elif place == "beside":
        ph["pos"] = (30.0, 10.0, 800.0)
    else:
        src["half_angle"] = 1e-9
        det.update(xmin=-1.0, xmax=1.0, ymin=-1.0, ymax=1.0)
    I = m.Instrument(ins)
    n = 100_003
    got, ref = I.run(n, seed=9)[0], I.run(n, seed=9, ledger=I.new_ledger())[0]
    torch_cuda.cuda.synchronize()
    assert int(ref["count"].sum()) > 1000
    assert np.array_equal(got["count"].cpu().numpy(), ref["count"].cpu().numpy())
    for k in ("sum_w", "sum_w2"):
        g, r = got[k].cpu().numpy(), ref[k].cpu().numpy()
        assert np.all(np.abs(g - r) <= 1e-11 * np.abs(r)), k
