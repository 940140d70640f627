"""Photons scattered once: plain runs walk the primary chords as a wave's bundle
(depth and interaction point), runs with a ledger event by event.  The same
photons interact in the same places up to the rounding of runs cut in two, so
counts agree (a photon within that rounding of a pixel's edge is not expected
among these) and sums within the parity bar.  Volumes and views of the bundle
walk's test; ray counts that leave the last wave partly filled, which takes the
event walk."""
import numpy as np
import pytest

import workloads

from test_gpu_bundle import VIEWS, VOLUMES, torch_cuda  # noqa: F401
from test_gpu_parity import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("view,aim", [(0, True), (1, True), (2, False), (3, True)])
@pytest.mark.parametrize("name", ["luggage 96", "noise 64x65x63", "one odd voxel", "shell 70", "slabs x 129", "thin plate"])
def test_scattered_once(torch_cuda, name, view, aim):  # noqa: F811
    import paper_2410_08747_amd as m
    angle, voxel, strata, n = VIEWS[view]
    announce("scattered once", name, VIEWS[view], aim)
    mu = workloads.make_scatter_tables(workloads.make_mu_tables(3))
    ins = workloads.edct_projection(VOLUMES[name](), mu, angle=angle, strata=strata, nx=16, ny=8, ne=4, scatter_order=1,
                                    aim=aim)
    ins["components"][1]["voxel"] = voxel
    if not aim:  # isotropic: a monitor that covers most of the forward half
        ins["components"][2].update(xmin=-4000.0, xmax=4000.0, ymin=-4000.0, ymax=4000.0)
    I = m.Instrument(ins)
    got, ref = I.run(n, seed=8)[0], I.run(n, seed=8, ledger=I.new_ledger())[0]
    torch_cuda.cuda.synchronize()
    assert int(ref["count"].sum()) > 100
    assert np.array_equal(got["count"].cpu().numpy(), ref["count"].cpu().numpy())
    for k in ("sum_w", "sum_w2"):
        g, r = got[k].cpu().numpy(), ref[k].cpu().numpy()
        assert np.all(np.abs(g - r) <= 1e-9 * np.abs(r)), (k, np.max(np.abs(g - r) / np.where(r != 0, r, 1)))
