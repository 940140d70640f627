"""The wave-wide walk of plain runs under the fixed-step model against the
step-by-step loop that runs with a ledger take: a layer of one material gives
it to the steps that end there, and only mixed layers are stepped through.  The
volumes, angles and strata are those of the exact model's test; the steps run
from a tenth of a voxel to two and a half (a last step then ends up to that far
behind the volume and reads the clamped voxel).  Counts equal; every step reads
the voxel that the loop reads, so sums differ by the rounding of runs cut in
two."""
import numpy as np
import pytest

import workloads

from test_gpu_bundle import VIEWS, VOLUMES, noise, torch_cuda  # noqa: F401
from test_gpu_parity import announce

pytestmark = pytest.mark.gpu


def check(torch, ins, n, seed):
    import paper_2410_08747_amd as m
    I = m.Instrument(ins)
    got, ref = I.run(n, seed=seed)[0], I.run(n, seed=seed, ledger=I.new_ledger())[0]
    torch.cuda.synchronize()
    assert int(ref["count"].sum()) > 1000
    assert np.array_equal(got["count"].cpu().numpy(), ref["count"].cpu().numpy())
    for k in ("sum_w", "sum_w2"):
        g, r = got[k].cpu().numpy(), ref[k].cpu().numpy()
        assert np.all(np.abs(g - r) <= 1e-11 * np.abs(r)), (k, np.max(np.abs(g - r) / np.where(r != 0, r, 1)))


@pytest.mark.parametrize("view,step", [(0, 1.0 / 3.0), (1, 0.1), (1, 2.5), (2, 0.75), (3, 1.7)])
@pytest.mark.parametrize("name", sorted(VOLUMES))
def test_bundle_of_steps_equals_the_step_loop(torch_cuda, name, view, step):  # noqa: F811
    angle, voxel, strata, n = VIEWS[view]
    announce("bundle of steps", name, VIEWS[view], step)
    ins = workloads.edct_projection(VOLUMES[name](), workloads.make_mu_tables(3), angle=angle, strata=strata, nx=64, ny=32,
                                    ne=4, step=step * voxel)
    ins["components"][1]["voxel"] = voxel
    check(torch_cuda, ins, n, 8)


@pytest.mark.parametrize("place", ["inside", "beside", "along the axis"])
def test_bundles_of_steps_from_other_places(torch_cuda, place):  # noqa: F811
    announce("bundle of steps", place)
    ins = workloads.edct_projection(noise((70, 72, 76), 5), workloads.make_mu_tables(3), angle=0.0, strata=32, nx=32, ny=16,
                                    ne=4, step=0.4)
    src, ph, det = ins["components"]
    if place == "inside":
        ph["pos"], src["half_angle"] = (3.0, -2.0, 5.0), 1.2
        det.update(pos=(0.0, 0.0, 60.0), xmin=-100.0, xmax=100.0, ymin=-100.0, ymax=100.0)
    elif place == "beside":
        ph["pos"] = (30.0, 10.0, 800.0)
    else:
        src["half_angle"] = 1e-9
        det.update(xmin=-1.0, xmax=1.0, ymin=-1.0, ymax=1.0)
    check(torch_cuda, ins, 100_003, 9)
